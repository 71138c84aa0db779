"""Collide adjoint across its launch shapes: 256, 512 and 1024 threads per
workgroup, velocity rows of whole quadruples and odd ones, grids whose nodes
exceed the registers that hold the incoming adjoint, and the FP64 fallback of
the sample sums.  Bar as in the other adjoint tests: a few FP32 ulps per term,
relative 1e-5 of each cell's largest value against the FP64 oracle.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    dict(nx=3, ny=3, nv=(8, 8, 8), vmax=3.5),        # 1024 threads: one cell per CU
    dict(nx=20, ny=20, nv=(8, 6, 4), vmax=3.5),      # 512: two cells per CU
    dict(nx=36, ny=30, nv=(6, 6, 8), vmax=3.0),      # 256: four cells per CU, grid walks twice
    dict(nx=36, ny=30, nv=(5, 7, 3), vmax=3.0),      # ... single nodes (odd rows)
    dict(nx=2, ny=2, nv=(22, 20, 20), vmax=5.0),     # 8800 nodes: past the registers of 1024 threads
    dict(nx=2, ny=2, nv=(20, 20, 21), vmax=5.0),     # 8400 nodes, odd rows
    dict(nx=2, ny=1, nv=(2, 1, 1), vmax=1.0),        # fewer nodes than the reduction scratch
]


def _lam(o, seed):
    w = o.node_weights()
    return w * np.random.default_rng(seed).standard_normal(o.shape)


@pytest.mark.parametrize("group", [0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_collide_adjoint_launch_shapes(oracle_mod, case, group):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(CASES[case], delta=10.0, eps=0.1, n_pairs=301, sample_group=group, bc=1, mix16=4)
    print("[gpu-case] collide adjoint shapes", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    h = (0.2 * np.random.default_rng(case).standard_normal(o.shape)).astype(np.float32)
    lo = _lam(o, 70 + case)
    corr = o.nv > 2
    ref = o.collide_adjoint(h.astype(np.float64), lo, 5, correction=corr).reshape(-1, o.nv)
    lo_d = torch.from_numpy(lo).cuda()
    g.collide_adjoint(torch.from_numpy(h).cuda(), lo_d, lo_d, 5, correction=corr)
    got = lo_d.cpu().numpy().reshape(-1, o.nv)
    bad = np.abs(got - ref).max(1) > 1e-5 * np.abs(ref).max(1)
    assert not bad.any(), np.flatnonzero(bad)[:10]


def test_collide_adjoint_beyond_fixed_point(oracle_mod):
    """Terms above 2^22 times the cell's scale (a rarefaction far outside the
    flow range, an adjoint not scaled by the weights): the FP64 sums."""
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(nx=2, ny=2, nv=12, vmax=4.5, delta=1.0e8, eps=0.1, n_pairs=500, dt=0.01, sample_group=0, bc=1, mix16=4)
    print("[gpu-case] collide adjoint fallback", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    rng = np.random.default_rng(3)
    h = (0.2 * rng.standard_normal(o.shape)).astype(np.float32)
    lo = rng.standard_normal(o.shape)
    # the samples do reach past the range
    idx, q = g.debug_pairs(0, 5, 0, 500)
    w = o.node_weights().reshape(-1)[: o.nv]
    l0 = lo.reshape(-1, o.nv)[0]
    keep = idx[:, 2] >= 0
    a, b, s, t = idx[keep].T
    lg = q[keep] * (l0[s] / w[s] + l0[t] / w[t] - l0[a] / w[a] - l0[b] / w[b])
    scale = 2.0 ** (np.floor(np.log2(np.abs(l0).max())) + 1)
    assert np.abs(lg).max() > 2.0 ** 22 * scale
    ref = o.collide_adjoint(h.astype(np.float64), lo, 5, correction=False).reshape(-1, o.nv)
    ls = g.empty_adjoint()
    g.collide_adjoint(torch.from_numpy(h).cuda(), torch.from_numpy(lo).cuda(), ls, 5, correction=False)
    got = ls.cpu().numpy().reshape(-1, o.nv)
    assert (np.abs(got - ref).max(1) <= 1e-5 * np.abs(ref).max(1)).all()
    assert g.read_status() == 0


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("kw", [
    dict(nx=17, ny=33, nv=(4, 4, 6), vmax=2.5, bc=0),     # ragged tiles (8 x 16 cells), pairs of velocities
    dict(nx=8, ny=16, nv=(6, 3, 8), vmax=(3.0, 2.0, 3.0), bc=0),   # exact tiles, v_y = 0 nodes
    dict(nx=9, ny=18, nv=(5, 4, 3), vmax=2.5, bc=0),      # odd rows: single velocities
    dict(nx=19, ny=17, nv=(4, 6, 4), vmax=2.5, bc=1),     # periodic wrap across tiles
])
def test_step_adjoint_tiles(oracle_mod, kw, offset):
    """Both sweeps in one pass, faces included, also with adjoint buffers that
    are 8-byte aligned only."""
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(kw, delta=5.0, eps=0.1, n_pairs=200, sample_group=0, order=2)
    print("[gpu-case] adjoint tiles", kw, offset, flush=True)
    g, o = pkg.Boltz(flags=pkg.WITH_ADJOINT, **kw), oracle_mod.Oracle(**kw)
    wk = dict(lid_u=0.1, tau_left=1.03, tau_right=0.98, tau_top=1.02,
              tau_bottom_x=1.0 + 0.05 * np.cos(np.arange(kw["nx"])))
    cavity = kw["bc"] == 0
    wg, wo = (pkg.Walls(**wk), oracle_mod.Walls(**wk)) if cavity else (None, None)
    h = (0.2 * np.random.default_rng(1).standard_normal(o.shape)).astype(np.float32)
    lam = _lam(o, 2)
    buf = torch.empty(2 * g.numel + 3, dtype=torch.float64, device="cuda")
    lo = buf[offset:offset + g.numel]
    li = buf[g.numel + 2 - offset:2 * g.numel + 2 - offset]
    lo.copy_(torch.from_numpy(lam).reshape(-1))
    grad = torch.zeros(g.grad_size(), dtype=torch.float64, device="cuda")
    g.step_adjoint(torch.from_numpy(h).cuda(), lo, li, grad, wg, 4)
    ref, ref_g = o.step_adjoint(h.astype(np.float64), lam, wo, 4)
    got = li.cpu().numpy().reshape(ref.shape)
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    if cavity:
        assert np.abs(grad.cpu().numpy() - ref_g).max() <= 1e-5 * np.abs(ref_g).max()
