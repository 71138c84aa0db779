// adjoint.hpp -- reverse mode of one time-split step on gfx950.
//
// The paper has no adjoint; every kernel here is the transpose of the
// linearisation of the forward kernel it names, for fixed Philox samples:
//   collide_adj_kernel  S3-S5 (forward recomputed per cell in LDS)
//   wall_adj_kernel     S1    adjoint of the face densities n_w and of the
//                             re-emitted ghosts, wall-parameter partials
//   stream_adj_kernel   S2    Beam-Warming sweeps transposed (order 2)
//   order1_adj_kernel   S2    first-order unsplit step transposed
//   lid_adj_kernel      S6    adjoint of the lid shear D
// Adjoints are FP64, cell-major like h.  Wall parameters theta are indexed
//   0 lid_u, 1 tau_left, 2 tau_right, 3 tau_top, 4 + ix: tau of bottom face ix.
#pragma once

#include "kernels.hpp"

namespace boltz {

// -------------------------------------------------------- collision --
// Adjoint of the gain/loss pass: lI is the adjoint of the increment of h
// (FP32 tile).  A sample adds dJ/dg (1 + eps h_b) to the adjoint of h_a and
// dJ/dg (1 + eps h_a) to that of h_b, with
// dJ/dg = k_a* lI_a* + k_b* lI_b* - k_a lI_a - k_b lI_b and the sample's own
// coefficients k (FP32 table records or the FP64 values of the draw).
// AdjFixed: the terms, divided by the cell's power-of-two scale S (inv_s =
// 1/S), go to 64-bit fixed-point accumulators as in the forward pass; a term
// outside [-win, win) S (or not finite) raises the flag: the cell's sums are
// then formed again by AdjF64, FP64 compare-and-swap adds.  A record adds at
// most two terms to one node, so win = min(2^18, 2^30 / N_t) keeps every sum
// below 2^31 S, the range of the accumulators, however the signs fall.
struct AdjFixed {
  unsigned long long* acc;
  double inv_s;
  unsigned* flag;
  unsigned win;
  __device__ __forceinline__ bool in_range(long long d) const {
    return (unsigned)((int)(d >> 32)) + win < 2u * win;
  }
  __device__ __forceinline__ void add(int a, int b, double lg, double fa, double fb) const {
    // both values first; straight-line adds when the whole wavefront has
    // them in range (a discarded sample adds 0)
    const double ks = lg * inv_s;
    const long long da = fixed_of(ks, fa), db = fixed_of(ks, fb);
    const bool ok = in_range(da) & in_range(db);
    if (__all(ok)) {
      __hip_atomic_fetch_add(&acc[a], (unsigned long long)da, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __hip_atomic_fetch_add(&acc[b], (unsigned long long)db, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else if (!ok) {
      *flag = 1u;  // (the other lanes' terms are dropped with the cell's sums)
    }
  }
};

struct AdjF64 {
  double* ls;
  __device__ __forceinline__ void add(int a, int b, double lg, double fa, double fb) const {
    if (lg != 0.0) {
      lds_add_f64(&ls[a], lg * fa);
      lds_add_f64(&ls[b], lg * fb);
    }
  }
};

template <int BLOCK, bool TABLE, int PU, class Acc>
__device__ __forceinline__ void gain_loss_adj(const Params& P, const TablesLDS& T, const float* hs,
                                              const float* lI, const Acc& A, uint32_t group, uint32_t step,
                                              const uint2* __restrict__ tidx,
                                              const float4* __restrict__ tcoef) {
  const int tid = threadIdx.x;
  const double eps = P.eps;
  const uint32_t nt = (uint32_t)P.n_pairs;
  if (TABLE) {
    const uint2* ri = tidx + (int64_t)group * nt;
    const float4* rk = tcoef + (int64_t)group * nt;
    // one pass: PU records per thread; in the masked (last) pass slots past
    // the end of the table load and add nothing
    auto pass = [&](uint32_t m0, uint32_t stride, const bool masked) {
      uint2 id[PU];
      float4 kk[PU];
      bool ok[PU];
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const uint32_t m = m0 + u * stride;
        ok[u] = !masked || m < nt;
        id[u] = ok[u] ? ri[m] : make_uint2(0u, 0u);
        kk[u] = ok[u] ? rk[m] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      // the six gathers of every record in flight together
      float l[PU][4], ha[PU], hb[PU];
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        const int a = (int)(id[u].x & 0xFFFFu), b = (int)(id[u].x >> 16);
        l[u][0] = lI[id[u].y & 0xFFFFu];
        l[u][1] = lI[id[u].y >> 16];
        l[u][2] = lI[a];
        l[u][3] = lI[b];
        ha[u] = hs[a];
        hb[u] = hs[b];
      }
#pragma unroll
      for (int u = 0; u < PU; ++u) {
        if (!ok[u]) continue;
        const double lg = fma((double)kk[u].x, (double)l[u][0], (double)kk[u].y * (double)l[u][1]) -
                          fma((double)kk[u].z, (double)l[u][2], (double)kk[u].w * (double)l[u][3]);
        A.add((int)(id[u].x & 0xFFFFu), (int)(id[u].x >> 16), lg, fma(eps, (double)hb[u], 1.0),
              fma(eps, (double)ha[u], 1.0));
      }
    };
    table_walk<BLOCK, PU>(nt, tid, false, pass);
  } else {
    for (uint32_t m = tid; m < nt; m += BLOCK) {
      const Pair p = sample_pair(P, T, group, step, m, nullptr);
      if (p.as >= 0) {
        const double lg = fma(p.kas, (double)lI[p.as], p.kbs * (double)lI[p.bs]) -
                          fma(p.ka, (double)lI[p.a], p.kb * (double)lI[p.b]);
        const double ha = (double)hs[p.a], hb = (double)hs[p.b];
        A.add(p.a, p.b, lg, fma(eps, hb, 1.0), fma(eps, ha, 1.0));
      }
    }
  }
}

// Dynamic LDS of the collide adjoint: the collide kernel's fixed-point layout
// (h^s tile, FP32 array, 64-bit accumulators), then the tables and the
// per-axis table of y . psi.  The block sums (25 doubles per wavefront) use
// the accumulators' region between the two pair passes.
__host__ __device__ inline size_t collide_adj_acc(int nv, int block) {
  const size_t a = ((size_t)nv * 8 + 15) & ~(size_t)15, r = (size_t)25 * (block / 64) * 8;
  return a > r ? a : ((r + 15) & ~(size_t)15);
}
__host__ __device__ inline size_t collide_adj_lds(int nv, int ns, bool sampler, int block) {
  return 2 * CollideLDS::tile(nv) + collide_adj_acc(nv, block) + TablesLDS::bytes(ns, sampler) + 8 * (size_t)ns;
}

// static LDS of the collide adjoint (maxima per wavefront, flag)
__host__ __device__ inline size_t collide_adj_static_lds(int block) { return 8 * (size_t)(block / 64) + 16; }

// Largest value over the wavefront, in every lane (no LDS traffic).
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_f64<kDppXor1>(v));
  v = fmax(v, dpp_f64<kDppXor2>(v));
  v = fmax(v, dpp_f64<kDppHalfMirror>(v));
  v = fmax(v, dpp_f64<kDppMirror>(v));
  const unsigned a = (unsigned)__double2loint(v), b = (unsigned)__double2hiint(v);
  const auto l = __builtin_amdgcn_permlane16_swap(a, a, false, false), h = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  v = fmax(__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1]));
  const unsigned c = (unsigned)__double2loint(v), d = (unsigned)__double2hiint(v);
  const auto m = __builtin_amdgcn_permlane32_swap(c, c, false, false), n = __builtin_amdgcn_permlane32_swap(d, d, false, false);
  return fmax(__hiloint2double((int)n[0], (int)m[0]), __hiloint2double((int)n[1], (int)m[1]));
}

// V consecutive values at p, which V = 4 finds on a 16-byte boundary (one or
// two 16-byte accesses, no bank conflicts between neighbouring lanes).
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <int V>
__device__ __forceinline__ void get_v(const float* p, float (&v)[V]) {
  if constexpr (V == 4) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    v[0] = p[0];
  }
}
template <int V>
__device__ __forceinline__ void put_v(float* p, const float (&v)[V]) {
  if constexpr (V == 4) *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
  else p[0] = v[0];
}
template <int V>
__device__ __forceinline__ void get_v(const unsigned long long* p, unsigned long long (&v)[V]) {
  if constexpr (V == 4) {
    const u64x2* q = reinterpret_cast<const u64x2*>(p);
    const u64x2 a = q[0], b = q[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  } else {
    v[0] = p[0];
  }
}
template <int V>
__device__ __forceinline__ void clear_v(unsigned long long* p) {
  if constexpr (V == 4) {
    u64x2* q = reinterpret_cast<u64x2*>(p);
    q[0] = u64x2{0ull, 0ull};
    q[1] = u64x2{0ull, 0ull};
  } else {
    p[0] = 0ull;
  }
}
// adjoint values in global memory (read once, written once)
template <int V>
__device__ __forceinline__ void load_lam(const double* p, double (&v)[V]) {
  if constexpr (V == 4) {
    const f64x2* q = reinterpret_cast<const f64x2*>(p);
    const f64x2 a = q[0], b = q[1];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  } else {
    v[0] = p[0];
  }
}
template <int V>
__device__ __forceinline__ void store_lam(double* p, const double (&v)[V]) {
  if constexpr (V == 4) {
    f64x2* q = reinterpret_cast<f64x2*>(p);
    __builtin_nontemporal_store(f64x2{v[0], v[1]}, &q[0]);
    __builtin_nontemporal_store(f64x2{v[2], v[3]}, &q[1]);
  } else {
    p[0] = v[0];
  }
}

// Reverse mode of collide_kernel: lo = adjoint of h^{n+1}, ls = adjoint of
// h^s (FP64; ls may equal lo, each node is read before it is written, by the
// thread that writes it).  Per cell the forward pass is recomputed in LDS
// (h^c and the correction's x); then with z_k = sum_j lo_j F^c_j psi_k / eps
// and M y = z,
//   lhc_j = lo_j (1 + x.psi_j) - eps w_j (y.psi_j)(x.psi_j)   (adjoint of h^c)
//   lI_j  = lhc_j - eps w_j (y.psi_j)      (adjoint of the increment of h)
// and ls = lhc plus the sample terms of gain_loss_adj.  Without the
// correction, or when M is not positive definite (status bit 1, as in the
// forward pass), x = y = 0.  LDS reuse: h^c is overwritten by lI (FP32), the
// forward's accumulators by the adjoint sums, 64-bit fixed point in units of
// S 2^-32 with S the power of two above the cell's max |lhc|.
//
// V consecutive nodes of one velocity row per thread and group (V = 4 where
// nv_z is a multiple of 4, else 1).  lo is read once, into 8 registers a
// thread while the forward pair loop runs, and becomes lhc there; the next
// cell's lo and h^s are requested in the last pass.  Bound by the LDS (two
// gathers and four adds, then six gathers and two adds per pair), then by
// the node passes' latency: one workgroup per CU on 20^3, so 1024 threads.
// 64x64 cavity, 20^3, 20 000 shared pairs, us per cell: 45.7 with 512
// threads, three reads of lo and per-node LDS accesses; now 37 (21.8 of them
// the two pair loops, 2.0 h^c, 1.3 + 1.6 sums and fold, 2.0 solves, 4.0
// adjoints, 4.5 output, staging and barrier).
constexpr int kAdjKeep = 8;  // lo values per thread kept in registers

template <int BLOCK, bool TABLE, int V>
__global__ __launch_bounds__(BLOCK, 4) void collide_adj_kernel(Params P, const float* __restrict__ hs_g,
                                                            const double* lo_g, double* ls_g, uint32_t step,
                                                            uint32_t flags, const uint2* __restrict__ tidx,
                                                            const float4* __restrict__ tcoef) {
  extern __shared__ __align__(16) unsigned char dsm[];
  __shared__ double mred[BLOCK / 64];
  __shared__ unsigned wide_flag;
  constexpr int NG = kAdjKeep / V;        // groups of V nodes kept per thread
  constexpr int NW = BLOCK / 64;
  const int nv = P.nv, n0 = P.n[0], n1 = P.n[1], n2 = P.n[2], ns = n0 + n1 + n2;
  const int ng = nv / V;                  // groups of the cell
  const int64_t ncells = (int64_t)P.nx * P.ny;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  float* hs = reinterpret_cast<float*>(dsm);
  float* accf = reinterpret_cast<float*>(dsm + CollideLDS::tile(nv));
  unsigned long long* acc64 = reinterpret_cast<unsigned long long*>(dsm + 2 * CollideLDS::tile(nv));
  double* lsh = reinterpret_cast<double*>(acc64);
  double* red = lsh;                      // block sums, between the pair passes
  unsigned char* tb = dsm + 2 * CollideLDS::tile(nv) + collide_adj_acc(nv, BLOCK);
  TablesLDS T;
  load_tables(P, tb, !TABLE, T);
  double* yt = reinterpret_cast<double*>(tb + TablesLDS::bytes(ns, !TABLE));
  const double* vx = T.v;
  const double* vy = T.v + n0;
  const double* vz = T.v + n0 + n1;
  const double* omx = T.om;
  const double* omy = T.om + n0;
  const double* omz = T.om + n0 + n1;
  const bool correct = !(flags & 1u);
  const double eps = P.eps;
  // this thread's index, hidden from the optimiser: the passes below form
  // their node indices from it, which otherwise stay in registers (hoisted out
  // of the cell loop) across the pair loops and spill
  auto here = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    return t;
  };
  // lo of this thread's groups; groups past the registers (i >= NG * BLOCK)
  // read theirs again in each pass
  double lam[NG][V];
  auto load_lo = [&](const double* lo) {
    const int t = here();
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      load_lam<V>(lo + min(t + g * BLOCK, ng - 1) * V, lam[g]);
    }
  };
  // h^s of the next cell waits in registers during the second pair loop
  constexpr int NR = prefetch_regs<BLOCK>();
  const int nv4 = nv >> 2;
  const bool pvec = V == 4 && nv4 <= NR * BLOCK && (reinterpret_cast<uintptr_t>(hs_g) & 15) == 0;
  Prefetch<NR> pre;
  auto stage = [&](const float* src) {
    if (pvec) {
      pre.store(hs, tid, BLOCK, nv4);
    } else {
      for (int j = tid; j < nv; j += BLOCK) hs[j] = src[j];
    }
  };
  // velocity row (jx, jy) and first z node of group i
  auto decode = [&](int i, int& jx, int& jy, int& jz) {
    const int row = div_small(i * V, n2);
    jz = i * V - row * n2;
    jx = div_small(row, n1);
    jy = row - jx * n1;
  };
  // adjoints of h^c (returned) and of the increment of the nodes of group i
  auto lam_group = [&](int i, const double (&l)[V], double (&lhc)[V], double (&lI)[V]) {
    if (!correct) {
#pragma unroll
      for (int e = 0; e < V; ++e) lhc[e] = lI[e] = l[e];
      return;
    }
    int jx, jy, jz;
    decode(i, jx, jy, jz);
    const double xa = T.xt[jx] + T.xt[n0 + jy], ya = yt[jx] + yt[n0 + jy], wa = omx[jx] * omy[jy];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const double xpsi = xa + T.xt[n0 + n1 + jz + e], ypsi = ya + yt[n0 + n1 + jz + e];
      const double ewy = eps * (wa * omz[jz + e]) * ypsi;
      lhc[e] = fma(l[e], xpsi, l[e]) - ewy * xpsi;
      lI[e] = lhc[e] - ewy;
    }
  };
  int64_t cell = blockIdx.x;
  if (cell < ncells) {
    if (pvec) pre.load(hs_g + cell * nv, tid, BLOCK, nv4);
    stage(hs_g + cell * nv);
  }
  for (int j = tid; j < nv; j += BLOCK) accf[j] = 0.0f;
  for (int j = tid; j < nv; j += BLOCK) acc64[j] = 0ull;
  for (; cell < ncells; cell += gridDim.x) {
    const double* lo = lo_g + cell * nv;
    load_lo(lo);
    __syncthreads();
    // ---- forward: increments and h^c, and the sums z
    const uint32_t group = (P.sample_group == 0) ? 0u : (uint32_t)(cell / P.sample_group);
    gain_loss<BLOCK, TABLE, ACC_FIXED, 2>(P, T, hs, accf, acc64, group, step, tidx, tcoef);
    __syncthreads();
    double zs[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    auto hc_group = [&](int i, const double (&l)[V]) {
      int jx, jy, jz;
      decode(i, jx, jy, jz);
      const double a = vx[jx], b = vy[jy];
      double us = 0.0, uz = 0.0, uzz = 0.0;
      float f[V], h[V];
      unsigned long long q[V];
      get_v<V>(accf + i * V, f);
      get_v<V>(hs + i * V, h);
      get_v<V>(acc64 + i * V, q);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const double dh = (double)f[e] + from_fixed(q[e]);
        f[e] = (float)((double)h[e] + dh);
        const double u = l[e] * fma(eps, (double)f[e], 1.0), c = vz[jz + e];
        us += u;
        uz += c * u;
        uzz += (c * c) * u;
      }
      put_v<V>(accf + i * V, f);
      zs[0] += us;
      zs[1] += a * us;
      zs[2] += b * us;
      zs[3] += uz;
      zs[4] += (a * a + b * b) * us + uzz;
    };
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int i = here() + g * BLOCK;
      if (i < ng) hc_group(i, lam[g]);
    }
    for (int i = tid + NG * BLOCK; i < ng; i += BLOCK) {
      double l[V];
      load_lam<V>(lo + i * V, l);
      hc_group(i, l);
    }
    if (correct) {
      __syncthreads();
      double acc[20];
      correction_sums<BLOCK>(T, P.zmom, hs, accf, n0, n1, n2, acc);
      const int rows = n0 * n1, nwd = rows >= BLOCK ? NW : (rows + 63) / 64;
      {
        const double z = wave_fold5(zs, lane);
        const int b5 = (lane >> 5) & 1, pos = 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1);
        if ((lane & 7) == 0 && pos < 3 - b5) red[(20 + 3 * b5 + pos) * NW + wid] = z;
        if (wid < nwd) {
          const double s = wave_fold20(acc, lane);
          const int b4 = (lane >> 4) & 1, b3 = (lane >> 3) & 1, b2 = (lane >> 2) & 1, b1 = (lane >> 1) & 1;
          const int p = 3 * b3 + 2 * b2 + b1;
          if (((lane & 1) == 0) && (b3 ? (b2 == 0) : (p < 3))) red[(10 * b5 + 5 * b4 + p) * NW + wid] = s;
        }
      }
      __syncthreads();
      // lo again (from cache), for the passes after the solve: kept across
      // the sums and the solve it would spill
      load_lo(lo);
      if (wid < 2) {
        // wavefront 0: M x = r, wavefront 1: M y = z; then x . psi, y . psi
        // per axis
        double t = 0.0;
        if (lane < 25)
          for (int w = 0; w < (lane < 20 ? nwd : NW); ++w) t += red[lane * NW + w];
        const const_f64* m0c = (const const_f64*)P.m0;
        const int rhs = __builtin_amdgcn_readfirstlane(wid);
        double M[15], r[5], x[5];
#pragma unroll
        for (int k = 0; k < 15; ++k) M[k] = m0c[k] + eps * lane_value(t, k);
#pragma unroll
        for (int k = 0; k < 5; ++k) r[k] = (rhs ? P.inv_eps : -eps) * lane_value(t, (rhs ? 20 : 15) + k);
        if (!solve5(M, r, x)) {
#pragma unroll
          for (int k = 0; k < 5; ++k) x[k] = 0.0;
          if (tid == 0) atomicOr(P.status, 1u);
        }
        double* tab = rhs ? yt : T.xt;
        for (int i = lane; i < ns; i += 64) {
          const double v = T.v[i], v2 = v * v;
          tab[i] = i < n0 ? x[1] * v + x[4] * v2 : (i < n0 + n1 ? x[2] * v + x[4] * v2 : x[0] + x[3] * v + x[4] * v2);
        }
      }
      __syncthreads();
    }
    // ---- adjoints of h^c (lam becomes lhc) and of the increment
    double scale = 1.0, inv_scale = 1.0;
    {
      double mx = 0.0;
      auto lI_group = [&](int i, double (&l)[V]) {
        double lhc[V], lI[V];
        lam_group(i, l, lhc, lI);
        float f[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
          f[e] = (float)lI[e];
          mx = fmax(mx, fabs(lhc[e]));
          l[e] = lhc[e];
        }
        put_v<V>(accf + i * V, f);
        clear_v<V>(acc64 + i * V);
      };
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int i = here() + g * BLOCK;
        if (i < ng) lI_group(i, lam[g]);
      }
      for (int i = tid + NG * BLOCK; i < ng; i += BLOCK) {
        double l[V];
        load_lam<V>(lo + i * V, l);
        lI_group(i, l);
      }
      // S = 2^e > max |lhc| of the cell (1 for an all-zero or non-finite cell)
      mx = wave_max(mx);
      if (lane == 0) mred[wid] = mx;
      if (tid == 0) wide_flag = 0u;
    }
    __syncthreads();
    {
      const double mx = lane_value(wave_max(lane < NW ? mred[lane] : 0.0), 0);
      if (mx > 0.0 && isfinite(mx)) {
        const int e = __builtin_amdgcn_frexp_exp(mx);  // mx = f 2^e, 1/2 <= f < 1
        scale = ldexp(1.0, e);
        inv_scale = ldexp(1.0, -e);
      }
    }
    const int64_t next = cell + gridDim.x;
    if (pvec && next < ncells) pre.load(hs_g + next * nv, tid, BLOCK, nv4);
    gain_loss_adj<BLOCK, TABLE, 2>(P, T, hs, accf, AdjFixed{acc64, inv_scale, &wide_flag, P.adj_win}, group, step, tidx, tcoef);
    __syncthreads();
    const bool wide = wide_flag != 0u;
    if (wide) {
      // (rare) a term beyond the fixed-point range: the sums in FP64
      __syncthreads();
      for (int j = tid; j < nv; j += BLOCK) lsh[j] = 0.0;
      __syncthreads();
      gain_loss_adj<BLOCK, TABLE, 1>(P, T, hs, accf, AdjF64{lsh}, group, step, tidx, tcoef);
      __syncthreads();
    }
    // ---- ls = lhc + the sums; the accumulators are left cleared and the
    // next cell's lo and h^s requested
    bool finite = true;
    double* dst = ls_g + cell * nv;
    auto out_group = [&](int i, const double (&lhc)[V]) {
      unsigned long long q[V];
      get_v<V>(acc64 + i * V, q);
      clear_v<V>(acc64 + i * V);
      float z[V];
      double v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
        v[e] = lhc[e] + (wide ? __longlong_as_double((long long)q[e]) : scale * from_fixed(q[e]));
        z[e] = 0.0f;
        finite = finite && isfinite(v[e]);
      }
      put_v<V>(accf + i * V, z);
      store_lam<V>(dst + i * V, v);
    };
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int i = here() + g * BLOCK;
      if (i < ng) out_group(i, lam[g]);
    }
    for (int i = tid + NG * BLOCK; i < ng; i += BLOCK) {
      double l[V], lhc[V], lI[V];
      load_lam<V>(lo + i * V, l);
      lam_group(i, l, lhc, lI);
      out_group(i, lhc);
    }
    if (next < ncells) stage(hs_g + next * nv);
    if (!finite) atomicOr(P.status, 2u);
  }
}

// ------------------------------------------------------------ walls --
__device__ __forceinline__ double face_tau(const Params& P, const WallArgs& W, int wall, int pos) {
  return wall == WALL_BOTTOM ? P.tau_b[pos] : W.tau[wall];
}

// Coefficients of the transposed Beam-Warming sweep of one node along one
// axis: li_i = a0 lo_i + a1 lo_{i+s} + a2 lo_{i+2s}, s the sign of v.
struct SweepAdj {
  double a0, a1, a2, C, an;
  int s;
  __device__ __forceinline__ SweepAdj(double v, double dt, double dl) {
    an = fabs(v);
    C = an * dt / dl;
    const double c2 = 0.5 * C * (1.0 - C);
    a0 = (1.0 - C) - c2;
    a1 = C + 2.0 * c2;
    a2 = -c2;
    s = v > 0.0 ? 1 : -1;
    if (v == 0.0) { a0 = 1.0; a1 = 0.0; a2 = 0.0; }
  }
};

// Adjoint of the gas-side face value (of an outgoing node of weight w) of
// face f of the wall a node with v != 0 leaves through: dJ/dn_w eps |v_n| w / D.
__device__ __forceinline__ double face_adj(const Params& P, const double* lnw, int f, double an, double w) {
  int wall, pos;
  face_of(P, f, wall, pos);
  return lnw[f] * P.eps * an * w / wall_consts(P, wall, pos)[1];
}

// Face term of the y sweep at (ix, iy) for a node leaving in y (order 2):
// hhat = h_a + (1 - C)(h_a - h_a')/2 at the two cells next to the wall.
__device__ __forceinline__ double y_face_term(const Params& P, const double* lnw, int ix, int iy, const SweepAdj& y,
                                              double w) {
  const int ia = y.s < 0 ? 0 : P.ny - 1, ib = y.s < 0 ? 1 : P.ny - 2;
  if (iy != ia && iy != ib) return 0.0;
  const double lh = face_adj(P, lnw, 2 * P.ny + (y.s < 0 ? 0 : P.nx) + ix, y.an, w);
  double t = 0.0;
  if (iy == ia) t += lh * (1.0 + 0.5 * (1.0 - y.C));
  if (iy == ib) t += -lh * 0.5 * (1.0 - y.C);
  return t;
}

// One workgroup per face f = f0 + (its index): lam is the adjoint of the
// output of the streaming pass that read the face's ghosts.  PHASE 0: lam as
// given (the y faces of order 2, every face of order 1); PHASE 1: the x faces
// of order 2, whose sweep's output is the y sweep's input, so lam is taken
// through the transposed y sweep (with the y faces' terms, whose lnw the
// launch before wrote) at the two cells next to the face.  For the incoming
// nodes (v . n > 0) the ghost h_w = (n_w R - 1)/eps enters the sweep with
// weight a1 + a2 at the adjacent cell and a2 at the next one (order 2: both
// ghost layers), or C (order 1); with lg_j its adjoint,
//   dJ/dn_w   = sum_in lg_j R_j / eps
//   dJ/dtheta = n_w sum_in lg_j dR_j/dtheta / eps
//               - dJ/dn_w (n_w / D) sum_in |v_n| w_j dR_j/dtheta,
// the last term from n_w = (A + eps B)/D, D = sum_in |v_n| w R (the sum over
// the mirror images of the outgoing nodes, which are the incoming ones).
// Writes lnw[f] and the partials gpart[2f] (lid velocity, top faces only)
// and gpart[2f + 1] (the face's temperature); grad: null, or the gradient
// (given to the last launch of a step).
// Latency bound: the incoming nodes only (a range of the normal axis), four
// per thread with their loads in flight together, 1024 threads (64x64 cavity,
// 20^3: 13 and 16 us a launch, 25..37 with 256 threads and one node at a time).
constexpr int kWallAdjBlock = 1024;

template <int PHASE>
__global__ __launch_bounds__(kWallAdjBlock) void wall_adj_kernel(Params P, WallArgs W, const double* __restrict__ lam,
                                                                 double* lnw, double* gpart, int f0, int nface,
                                                                 int per_xcd, double* grad) {
  __shared__ double red[5 * (kWallAdjBlock / 64)];
  __shared__ unsigned flag;
  int f = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (f >= nface) return;
  f += f0;
  int wall, pos;
  face_of(P, f, wall, pos);
  const int nx = P.nx, ny = P.ny, nv = P.nv, n1 = P.n[1], n2 = P.n[2];
  const int nax = (wall <= WALL_RIGHT) ? 0 : 1;
  const int sgn = (wall == WALL_LEFT || wall == WALL_BOTTOM) ? 1 : -1;
  int ax_, ay_, bx_, by_;
  switch (wall) {
    case WALL_LEFT: ax_ = 0; ay_ = pos; bx_ = 1; by_ = pos; break;
    case WALL_RIGHT: ax_ = nx - 1; ay_ = pos; bx_ = nx - 2; by_ = pos; break;
    case WALL_BOTTOM: ax_ = pos; ay_ = 0; bx_ = pos; by_ = 1; break;
    default: ax_ = pos; ay_ = ny - 1; bx_ = pos; by_ = ny - 2; break;
  }
  const double* la = lam + cell_off(P, ax_, ay_);
  const double* lb = lam + cell_off(P, bx_, by_);
  const double* R = ratio_row(P, wall, pos);
  const double dl = nax ? P.dy : P.dx;
  const double U = (wall == WALL_TOP) ? W.lid_u : 0.0;
  const double tau = face_tau(P, W, wall, pos);
  const bool periodic = P.bc == 1;
  const int64_t rowstep = (int64_t)nx * nv;
  // incoming nodes: v > 0 at the left / bottom wall, v < 0 at the others
  const int i0 = sgn > 0 ? P.vpos[nax] : 0, i1 = sgn > 0 ? P.n[nax] : P.vneg[nax];
  const int c0 = nax ? P.n[0] : i1 - i0, c1 = nax ? i1 - i0 : n1, nt = c0 * c1 * n2;
  double s[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  constexpr int NU = PHASE == 1 ? 2 : 4;  // nodes per thread and pass
  if (nt > 0) {
    NodeWalk walk((int)threadIdx.x, kWallAdjBlock, c1, n2);
    for (int tb = threadIdx.x; tb < nt; tb += NU * kWallAdjBlock) {
      double va[NU], vb[NU], Rj[NU], a1[NU], a2[NU], b1[NU], b2[NU];
      int jxs[NU], jys[NU], jzs[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const bool in = tb + u * kWallAdjBlock < nt;
        jxs[u] = in ? walk.jx + (nax ? 0 : i0) : 0;
        jys[u] = in ? walk.jy + (nax ? i0 : 0) : 0;
        jzs[u] = in ? walk.jz : 0;
        walk.next();
        const int j = (jxs[u] * n1 + jys[u]) * n2 + jzs[u];
        va[u] = la[j];
        vb[u] = P.order == 2 ? lb[j] : 0.0;
        Rj[u] = R[j];
        a1[u] = a2[u] = b1[u] = b2[u] = 0.0;
        if (PHASE == 1) {
          // the two cells downstream in y of each (zero beyond a wall; only
          // cavities have faces)
          const int sy = jys[u] < P.vneg[1] ? -1 : 1;
          const int y1 = pos + sy, y2 = pos + 2 * sy;
          const bool in1 = y1 >= 0 && y1 < ny, in2 = y2 >= 0 && y2 < ny;
          if (in1) { a1[u] = la[j + sy * rowstep]; b1[u] = lb[j + sy * rowstep]; }
          if (in2) { a2[u] = la[j + 2 * sy * rowstep]; b2[u] = lb[j + 2 * sy * rowstep]; }
        }
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (tb + u * kWallAdjBlock >= nt) continue;
        const int jx = jxs[u], jy = jys[u], jz = jzs[u];
        const double v1 = P.vtab[jx], v2 = P.vtab[kMaxAxis + jy], v3 = P.vtab[2 * kMaxAxis + jz];
        const double w = (P.omtab[jx] * P.omtab[kMaxAxis + jy]) * P.omtab[2 * kMaxAxis + jz];
        double xa = va[u], xb = vb[u];
        if (PHASE == 1) {
          const SweepAdj y(v2, P.dt, P.dy);
          xa = fma(y.a0, xa, fma(y.a1, a1[u], y.a2 * a2[u]));
          xb = fma(y.a0, xb, fma(y.a1, b1[u], y.a2 * b2[u]));
          if (!periodic && v2 != 0.0) {
            xa += y_face_term(P, lnw, ax_, pos, y, w);
            xb += y_face_term(P, lnw, bx_, pos, y, w);
          }
        }
        const double an = fabs(nax ? v2 : v1);
        const double C = an * P.dt / dl;
        double lg;
        if (P.order == 2) {
          const double c2 = 0.5 * C * (1.0 - C);
          lg = ((C + 2.0 * c2) + -c2) * xa + -c2 * xb;
        } else {
          lg = C * xa;
        }
        double dU, dT;
        wall_ratio_grad(Rj[u], v1, v2, v3, U, tau, dU, dT);
        const double aw = an * w;
        s[0] += lg * Rj[u];
        s[1] += lg * dU;
        s[2] += lg * dT;
        s[3] += aw * dU;
        s[4] += aw * dT;
      }
    }
  }
  block_sum<5>(s, red);
  if (threadIdx.x == 0) {
    const double nw = P.nw[f];
    const double D = wall_consts(P, wall, pos)[1];
    const double l = s[0] * P.inv_eps;
    const double q = l * nw / D;
    lnw[f] = l;
    publish(&gpart[2 * f], (wall == WALL_TOP) ? nw * s[1] * P.inv_eps - q * s[3] : 0.0);
    publish(&gpart[2 * f + 1], nw * s[2] * P.inv_eps - q * s[4]);
  }
  // the last workgroup of the last launch adds every face's partials to the
  // gradient in a fixed order: wavefront w the wall parameter w (lid velocity
  // from the top faces, temperatures of the left, right and top walls), then
  // one entry per bottom face
  if (grad && last_workgroup(P.count + 1, (uint32_t)nface, &flag)) {
    const int w = (int)threadIdx.x >> 6;
    if (w < 4) {
      const int first = w == 1 ? 1 : (w == 2 ? 2 * ny + 1 : 2 * (2 * ny + nx) + (w == 3 ? 1 : 0));
      const double t = wave_sum_of(gpart + first, nullptr, (w == 0 || w == 3) ? nx : ny, 2);
      if ((threadIdx.x & 63) == 0) grad[w] += t;
    }
    for (int i = threadIdx.x; i < nx; i += kWallAdjBlock)
      grad[4 + i] +=
          __hip_atomic_load(&gpart[2 * (2 * ny + i) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------- streaming --
// Transposed Beam-Warming step of order 2, y sweep then x sweep, in one pass
// over memory (out_i = a0 in_i + a1 in_{i-s} + a2 in_{i-2s} along an axis
// gives li_i = a0 lo_i + a1 lo_{i+s} + a2 lo_{i+2s}, over the downstream cells
// inside the cavity, wrapped when periodic; the ghost terms were taken by
// wall_adj_kernel), plus, at the two cells next to each wall, the adjoint of
// that wall's face density through the gas-side face value of its outgoing
// nodes.  One workgroup: kATX x kATY cells and 16 velocities (128 B a cell),
// staged with their downstream halo in LDS; a thread owns V velocities of one
// row of cells, forms the y-swept values of its row's columns (two halo
// columns included) in registers and applies the x sweep from that window,
// the same sums in the same order as one sweep after the other.  V = 2 where
// nv_z is even (a pair then shares its signs and coefficients), else 1.
// HBM bound: 16 B a node against 32 for two sweeps (64x64 cavity, 20^3:
// 147 us, 3.6 TB/s; 94 + 107 us before).  Workgroup order as in stream4.
constexpr int kATX = 8, kATY = 16, kAJ = 16;

__host__ __device__ inline int stream_adj_group(int nv) {
  const int nchunks = (nv + kAJ - 1) / kAJ;
  return nchunks < kChunkGroup ? nchunks : kChunkGroup;
}
__host__ __device__ inline int64_t stream_adj_units(int nx, int ny, int nv) {
  const int64_t tiles = (int64_t)((nx + kATX - 1) / kATX) * ((ny + kATY - 1) / kATY);
  const int cg = stream_adj_group(nv);
  return tiles * (((nv + kAJ - 1) / kAJ + cg - 1) / cg) * cg;
}

template <int V>
struct VecD {
  double e[V];
};
template <int V>
__device__ __forceinline__ VecD<V> load_vd(const double* p) {
  VecD<V> r;
  if constexpr (V == 2) {
    const f64x2 t = *reinterpret_cast<const f64x2*>(p);
    r.e[0] = t.x;
    r.e[1] = t.y;
  } else {
    r.e[0] = p[0];
  }
  return r;
}
template <int V>
__device__ __forceinline__ void store_vd(double* p, const VecD<V>& v) {
  if constexpr (V == 2) *reinterpret_cast<f64x2*>(p) = f64x2{v.e[0], v.e[1]};
  else p[0] = v.e[0];
}
template <int V>
__device__ __forceinline__ VecD<V> sweep3(const SweepAdj& c, const VecD<V>& x0, const VecD<V>& x1,
                                          const VecD<V>& x2) {
  VecD<V> r;
#pragma unroll
  for (int e = 0; e < V; ++e) r.e[e] = fma(c.a0, x0.e[e], fma(c.a1, x1.e[e], c.a2 * x2.e[e]));
  return r;
}

template <int V>
__global__ __launch_bounds__(kATY * (kAJ / V)) void stream_adj_kernel(Params P, const double* __restrict__ lo,
                                                                      double* __restrict__ li,
                                                                      const double* __restrict__ lnw, int tiles_x,
                                                                      int tiles_y, int nunits, int per_xcd) {
  constexpr int Q = kAJ / V, NT = kATY * Q, AX = kATX + 4, AY = kATY + 4;
  __shared__ __align__(16) double A[AY * AX * kAJ];
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= nunits) return;
  const int nx = P.nx, ny = P.ny, nv = P.nv, n1 = P.n[1], n2 = P.n[2];
  const int gsz = stream_adj_group(nv), per_group = tiles_x * tiles_y * gsz;
  const int cg = unit / per_group, rem = unit - cg * per_group;
  const int tile = rem / gsz, chunk = cg * gsz + (rem - tile * gsz);
  if (chunk * kAJ >= nv) return;  // padding unit of the last group
  const int ix0 = (tile % tiles_x) * kATX, iy0 = (tile / tiles_x) * kATY, j0 = chunk * kAJ;
  const bool periodic = P.bc == 1;
  // downstream sides that the chunk's velocities need (jx, and within one jx
  // also jy, increase with j)
  int fx, fy, fz, lx, ly, lz;
  node_decode(j0, n1, n2, fx, fy, fz);
  node_decode(min(j0 + kAJ, nv) - 1, n1, n2, lx, ly, lz);
  const bool oneX = fx == lx;
  const bool needR = P.vtab[lx] > 0.0, needL = P.vtab[fx] < 0.0;
  const bool needT = !oneX || P.vtab[kMaxAxis + ly] > 0.0, needB = !oneX || P.vtab[kMaxAxis + fy] < 0.0;
  const int c_lo = needL ? 0 : 2, c_hi = needR ? AX : AX - 2;
  const int r_lo = needB ? 0 : 2, r_hi = needT ? AY : AY - 2;
  const int q = threadIdx.x % Q, jq = j0 + V * q;
  {
    // all loads of a thread are issued before its LDS stores
    constexpr int kRows = NT / Q, kIter = (AY * AX + kRows - 1) / kRows;
    VecD<V> v[kIter];
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
      const int cidx = (int)threadIdx.x / Q + it * kRows;
#pragma unroll
      for (int e = 0; e < V; ++e) v[it].e[e] = 0.0;
      if (cidx >= AY * AX) continue;
      const int r = cidx / AX, c = cidx - r * AX;
      if (r < r_lo || r >= r_hi || c < c_lo || c >= c_hi || jq >= nv) continue;
      const int iy = iy0 - 2 + r, ix = ix0 - 2 + c;
      if (periodic) v[it] = load_vd<V>(lo + cell_off(P, wrapi(ix, nx), wrapi(iy, ny)) + jq);
      else if (ix >= 0 && ix < nx && iy >= 0 && iy < ny) v[it] = load_vd<V>(lo + cell_off(P, ix, iy) + jq);
    }
#pragma unroll
    for (int it = 0; it < kIter; ++it) {
      const int cidx = (int)threadIdx.x / Q + it * kRows;
      if (cidx < AY * AX) store_vd<V>(&A[cidx * kAJ + V * q], v[it]);
    }
  }
  const int r = (int)threadIdx.x / Q, iy = iy0 + r;
  const bool ok = jq < nv && iy < ny;
  int jx = 0, jy = 0;
  if (jq < nv) {
    const int row = div_small(jq, n2);
    jx = div_small(row, n1);
    jy = row - jx * n1;
  }
  const double vx = P.vtab[jx], vy = P.vtab[kMaxAxis + jy];
  const SweepAdj sx(vx, P.dt, P.dx), sy(vy, P.dt, P.dy);
  double w[V];
#pragma unroll
  for (int e = 0; e < V; ++e)
    w[e] = (P.omtab[jx] * P.omtab[kMaxAxis + jy]) * P.omtab[2 * kMaxAxis + (jq < nv ? jq + e - (jx * n1 + jy) * n2 : 0)];
  __syncthreads();
  if (!ok) return;
  // rows next to the wall that the node leaves through in y
  const bool yface = !periodic && vy != 0.0 && (sy.s < 0 ? iy <= 1 : iy >= ny - 2);
  VecD<V> t[AX];
#pragma unroll
  for (int c = 0; c < AX; ++c) {
#pragma unroll
    for (int e = 0; e < V; ++e) t[c].e[e] = 0.0;
    if (c < c_lo || c >= c_hi) continue;
    const int ix = ix0 - 2 + c;
    if (!periodic && (ix < 0 || ix >= nx)) continue;
    const double* col = &A[((r + 2) * AX + c) * kAJ + V * q];
    t[c] = sweep3<V>(sy, load_vd<V>(col), load_vd<V>(col + sy.s * AX * kAJ), load_vd<V>(col + 2 * sy.s * AX * kAJ));
    if (yface) {
#pragma unroll
      for (int e = 0; e < V; ++e) t[c].e[e] += y_face_term(P, lnw, ix, iy, sy, w[e]);
    }
  }
  // the wall that the node leaves through in x
  const bool xface = !periodic && vx != 0.0;
  const int ia = sx.s < 0 ? 0 : nx - 1, ib = sx.s < 0 ? 1 : nx - 2;
#pragma unroll
  for (int c = 0; c < kATX; ++c) {
    const int ix = ix0 + c;
    if (ix >= nx) break;
    VecD<V> x1, x2;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      x1.e[e] = sx.s > 0 ? t[c + 3].e[e] : t[c + 1].e[e];
      x2.e[e] = sx.s > 0 ? t[c + 4].e[e] : t[c].e[e];
    }
    VecD<V> o = sweep3<V>(sx, t[c + 2], x1, x2);
    if (xface && (ix == ia || ix == ib)) {
      const int f = (sx.s < 0 ? 0 : ny) + iy;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        const double lh = face_adj(P, lnw, f, sx.an, w[e]);
        if (ix == ia) o.e[e] += lh * (1.0 + 0.5 * (1.0 - sx.C));
        if (ix == ib) o.e[e] += -lh * 0.5 * (1.0 - sx.C);
      }
    }
    double* dst = li + cell_off(P, ix, iy) + jq;
    if constexpr (V == 2) __builtin_nontemporal_store(f64x2{o.e[0], o.e[1]}, reinterpret_cast<f64x2*>(dst));
    else dst[0] = o.e[0];
  }
}

// Transposed first-order unsplit step:
//   li = (1 - Cx - Cy) lo + Cx lo(downstream in x) + Cy lo(downstream in y)
// plus, at the cell next to each wall, dJ/dn_w eps |v_n| w_j / D for the
// wall's outgoing nodes (face value = the adjacent cell).  One thread per
// (cell, node).
constexpr int kOrder1AdjBlock = 256;

__global__ __launch_bounds__(kOrder1AdjBlock) void order1_adj_kernel(Params P, const double* __restrict__ lo,
                                                                     double* __restrict__ li,
                                                                     const double* __restrict__ lnw, int nchunks) {
  const int64_t cell = blockIdx.x / nchunks;
  const int chunk = blockIdx.x - (int)(cell * nchunks);
  const int nv = P.nv, n1 = P.n[1], n2 = P.n[2], nx = P.nx, ny = P.ny;
  const int j = chunk * kOrder1AdjBlock + threadIdx.x;
  if (j >= nv) return;
  int jx, jy, jz;
  node_decode(j, n1, n2, jx, jy, jz);
  const int ix = (int)(cell % nx), iy = (int)(cell / nx);
  const double vx = P.vtab[jx], vy = P.vtab[kMaxAxis + jy];
  const double Cx = fabs(vx) * P.dt / P.dx, Cy = fabs(vy) * P.dt / P.dy;
  const bool periodic = P.bc == 1;
  const int64_t o = cell * nv + j;
  double out = ((1.0 - Cx) - Cy) * lo[o];
  const double w = (P.omtab[jx] * P.omtab[kMaxAxis + jy]) * P.omtab[2 * kMaxAxis + jz];
  for (int ax = 0; ax < 2; ++ax) {
    const double v = ax == 0 ? vx : vy;
    if (v == 0.0) continue;
    const int s = v > 0.0 ? 1 : -1;
    const int n = ax == 0 ? nx : ny;
    const int i = (ax == 0 ? ix : iy) + s;
    const double Cv = ax == 0 ? Cx : Cy;
    if (i >= 0 && i < n) {
      out += Cv * lo[(ax == 0 ? cell_off(P, i, iy) : cell_off(P, ix, i)) + j];
    } else if (periodic) {
      const int iw = wrapi(i, n);
      out += Cv * lo[(ax == 0 ? cell_off(P, iw, iy) : cell_off(P, ix, iw)) + j];
    }
    // a cell next to the wall that this node leaves through
    const int ib = (ax == 0 ? ix : iy);
    if (!periodic && ((s < 0 && ib == 0) || (s > 0 && ib == n - 1))) {
      const int f = (ax == 0 ? (s < 0 ? 0 : ny) + iy : 2 * ny + (s < 0 ? 0 : nx) + ix);
      int wall, pos;
      face_of(P, f, wall, pos);
      out += lnw[f] * P.eps * fabs(v) * w / wall_consts(P, wall, pos)[1];
    }
  }
  li[o] = out;
}

// ---------------------------------------------------------- lid shear --
// Adjoint of weight * D, D = -(1/nx) sum over lid faces of 2 sum_j w_j v_x v_y
// hhat_j with hhat the gas-side value of the top cell for v_y > 0 and the
// wall emission with the first-order face density n_w = (A + eps B) / D for
// v_y < 0.  One workgroup per top face adds its part to lam (top cells, v_y > 0
// nodes; it depends on the walls alone, through the sums wlid) and, with grad,
// forms B of its face; the last workgroup adds the faces to grad[0] (lid
// velocity) and grad[3] (lid temperature).  Latency bound: the v_y > 0 nodes
// only, four in flight per thread.
constexpr int kLidAdjBlock = 1024;

__global__ __launch_bounds__(kLidAdjBlock) void lid_adj_kernel(Params P, const float* __restrict__ h, double weight,
                                                               double* __restrict__ lam, double* gpart,
                                                               double* grad) {
  __shared__ double red[kLidAdjBlock / 64];
  __shared__ unsigned flag;
  const int ix = blockIdx.x;
  const int n1 = P.n[1], n2 = P.n[2];
  const double c0 = weight * (-2.0 / P.nx);
  const double* k = wall_consts(P, WALL_TOP, ix);
  const double D = k[1], l = c0 * P.wlid[1] * P.inv_eps, le = l * P.eps / D;
  double* dst = lam + cell_off(P, ix, P.ny - 1);
  const float* src = h + cell_off(P, ix, P.ny - 1);
  const int i0 = P.vpos[1], c1 = n1 - i0, nt = P.n[0] * c1 * n2;
  double b[1] = {0.0};
  constexpr int NU = 4;
  if (nt > 0) {
    NodeWalk walk((int)threadIdx.x, kLidAdjBlock, c1, n2);
    for (int tb = threadIdx.x; tb < nt; tb += NU * kLidAdjBlock) {
      int js[NU], jxs[NU], jys[NU], jzs[NU];
      double old[NU];
      float hv[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const bool in = tb + u * kLidAdjBlock < nt;
        jxs[u] = in ? walk.jx : 0;
        jys[u] = in ? walk.jy + i0 : i0;
        jzs[u] = in ? walk.jz : 0;
        walk.next();
        js[u] = (jxs[u] * n1 + jys[u]) * n2 + jzs[u];
        old[u] = dst[js[u]];
        hv[u] = grad ? src[js[u]] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if (tb + u * kLidAdjBlock >= nt) continue;
        const double v1 = P.vtab[jxs[u]], v2 = P.vtab[kMaxAxis + jys[u]];
        const double w = (P.omtab[jxs[u]] * P.omtab[kMaxAxis + jys[u]]) * P.omtab[2 * kMaxAxis + jzs[u]];
        dst[js[u]] = old[u] + (c0 * w * v1 * v2 + le * v2 * w);
        b[0] += v2 * w * (double)hv[u];
      }
    }
  }
  if (!grad) return;
  block_sum<1>(b, red);
  if (threadIdx.x == 0) {
    const double nwt = (k[0] + P.eps * b[0]) / D, q = l * nwt / D;
    publish(&gpart[2 * ix], nwt * (c0 * P.wlid[2]) * P.inv_eps - q * P.wlid[4]);
    publish(&gpart[2 * ix + 1], nwt * (c0 * P.wlid[3]) * P.inv_eps - q * P.wlid[5]);
  }
  if (last_workgroup(P.count + 2, (uint32_t)P.nx, &flag) && threadIdx.x < 64) {
    const double su = wave_sum_of(gpart, nullptr, P.nx, 2), st = wave_sum_of(gpart + 1, nullptr, P.nx, 2);
    if (threadIdx.x == 0) {
      grad[0] += su;
      grad[3] += st;
    }
  }
}

}  // namespace boltz
