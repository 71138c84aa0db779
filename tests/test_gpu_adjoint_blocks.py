"""Workgroup sizes of the collide adjoint: both sides of the lines of the rule
(one, two and four cells per CU, few and many own pairs), in place, against the
FP64 oracle.  Bar of the adjoint tests: 1e-5 of each cell's largest value.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [0, 1])
@pytest.mark.parametrize("kw", [
    dict(nx=8, ny=6, nv=(8, 6, 4), vmax=3.5, n_pairs=2047),     # one cell a CU
    dict(nx=8, ny=6, nv=(8, 6, 4), vmax=3.5, n_pairs=2048),
    dict(nx=8, ny=6, nv=(8, 7, 5), vmax=3.5, n_pairs=2048),     # ... odd rows
    dict(nx=257, ny=1, nv=(8, 6, 4), vmax=3.5, n_pairs=301),    # two cells a CU
    dict(nx=257, ny=3, nv=(8, 6, 4), vmax=3.5, n_pairs=301),    # four
])
def test_collide_adjoint_block_rule(oracle_mod, kw, group):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(kw, delta=10.0, eps=0.1, sample_group=group, bc=1, mix16=4)
    print("[gpu-case] collide adjoint blocks", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    h = (0.2 * np.random.default_rng(4).standard_normal(o.shape)).astype(np.float32)
    lo = o.node_weights() * np.random.default_rng(5).standard_normal(o.shape)
    ref = o.collide_adjoint(h.astype(np.float64), lo, 5).reshape(-1, o.nv)
    lo_d = torch.from_numpy(lo).cuda()
    g.collide_adjoint(torch.from_numpy(h).cuda(), lo_d, lo_d, 5)
    got = lo_d.cpu().numpy().reshape(-1, o.nv)
    assert (np.abs(got - ref).max(1) <= 1e-5 * np.abs(ref).max(1)).all()
    assert g.read_status() == 0
