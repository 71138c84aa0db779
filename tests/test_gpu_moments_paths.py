"""Moments and lid shear on every path of the kernel (cells staged in LDS, rows
read in place: odd rows, states that are 4-byte aligned only, cells beyond the
staging buffer), repeated calls included.  FP64 sums of FP32 values on both
sides: 1e-11 of the largest value (summation order only), 1e-9 for the lid
shear, whose re-emitted part is a difference of sums 1/eps larger.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    dict(nx=9, ny=7, nv=(8, 8, 8), vmax=3.5),
    dict(nx=65, ny=3, nv=(6, 5, 12), vmax=3.0),      # more faces than a wavefront
    dict(nx=5, ny=4, nv=(7, 5, 9), vmax=3.0),        # odd rows
    dict(nx=3, ny=2, nv=(24, 24, 24), vmax=5.0),     # several pieces per thread
    dict(nx=2, ny=2, nv=(26, 26, 24), vmax=5.0),     # beyond the staging buffer
]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_moments_paths(oracle_mod, case, offset):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(CASES[case], delta=5.0, eps=0.1, n_pairs=10, mix16=16)
    print("[gpu-case] moments", kw, offset, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    h = (0.3 * np.random.default_rng(case).standard_normal(o.shape)).astype(np.float32)
    buf = torch.empty(g.numel + 4, dtype=torch.float32, device="cuda")
    hd = buf[offset:offset + g.numel]
    hd.copy_(torch.from_numpy(h).reshape(-1))
    mom = torch.empty(g.ncells * 11, dtype=torch.float64, device="cuda")
    D = torch.empty(1, dtype=torch.float64, device="cuda")
    for lid_u in (0.1, 0.2, 0.2):
        wk = dict(lid_u=lid_u, tau_left=1.02, tau_top=0.97)
        g.moments(hd, mom, pkg.Walls(**wk), D)
        ref, ref_d = o.moments(h.astype(np.float64), oracle_mod.Walls(**wk), lid_shear=True)
        got = mom.cpu().numpy().reshape(-1, 11)
        ref = np.asarray(ref).reshape(-1, 11)
        assert np.abs(got - ref).max() <= 1e-11 * np.abs(ref).max()
        assert abs(float(D) - ref_d) <= 1e-9 * abs(ref_d)
