"""Shared records rearranged by their first node (problems of many
record-cells): full and partial blocks of 4096 records, several sample groups,
both layouts that use them, the step's face launches, batches.  Bar of the
collision tests: 1e-5 of each cell's largest value against the FP64 oracle (FP32
state and coefficients, a few ulps per term).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# record-cells >= 6e7 and >= 512 cells a group select the grouped form
CASES = [
    dict(nx=64, ny=32, nv=(6, 6, 8), vmax=3.0, n_pairs=32768, sample_group=0),          # whole blocks
    dict(nx=60, ny=35, nv=(6, 6, 8), vmax=3.0, n_pairs=29999, sample_group=0),          # partial block, masked tail
    dict(nx=64, ny=64, nv=(8, 6, 4), vmax=3.0, n_pairs=20481, sample_group=2048),       # two groups
    dict(nx=60, ny=35, nv=(5, 7, 3), vmax=3.0, n_pairs=30001, sample_group=0, flags=4),  # odd rows, continuous pairs
    dict(nx=40, ny=40, nv=(22, 24, 24), vmax=5.0, n_pairs=40001, sample_group=0),       # partial-tile layout
]


def _cells(o, n=12):
    return np.unique(np.random.default_rng(1).integers(0, o.nx * o.ny, n))


@pytest.mark.parametrize("case", range(len(CASES)))
def test_collide_grouped_records(oracle_mod, case):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(CASES[case], delta=10.0, eps=0.1, bc=1, mix16=4)
    print("[gpu-case] grouped records", kw, flush=True)
    g = pkg.Boltz(**kw)
    assert g.ncells * g.n_pairs >= 6.0e7
    rng = np.random.default_rng(case)
    shape = (g.ny, g.nx, g.nv)
    h = (0.2 * rng.standard_normal(shape)).astype(np.float32)
    hd = torch.from_numpy(h).cuda()
    out = g.empty()
    g.collide(hd, out, 7)
    got = out.cpu().numpy().reshape(-1, g.nv)
    # the oracle on a few cells of each sample group: a problem of those cells
    # alone with the same pairs (sample_group 0 draws group 0's stream)
    per = kw["sample_group"] or g.ncells
    cells = [c for c in _cells(g) if c < per]
    o = oracle_mod.Oracle(**dict(kw, nx=len(cells), ny=1, sample_group=0, dt=g.dt, flags=kw.get("flags", 0) | 1))
    ref = o.collide(h.reshape(-1, g.nv)[cells].astype(np.float64).reshape(o.shape), 7).reshape(-1, g.nv)
    err = np.abs(got[cells] - ref).max(1)
    assert (err <= 1e-5 * np.abs(ref).max(1)).all(), err / np.abs(ref).max(1)
    # in place, without allocation, and as part of a cavity step: the same cells
    g.collide_noalloc(hd, hd, 7)
    assert np.array_equal(hd.cpu().numpy().reshape(-1, g.nv), got)
    assert g.read_status() == 0


@pytest.mark.parametrize("order", [1, 2])
def test_step_grouped_records(order):
    """The step draws and groups its records in the face launches: equal to
    streaming and colliding one after the other."""
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(nx=60, ny=35, nv=(6, 6, 8), vmax=3.0, n_pairs=29999, sample_group=0, delta=10.0, eps=0.1, order=order)
    g = pkg.Boltz(**kw)
    w = pkg.Walls(lid_u=0.1, tau_left=1.02)
    h = torch.randn(g.shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)) * 0.2
    a, b = g.empty(), g.empty()
    g.step(h, a, w, 3)
    g.stream(h, b, w)
    g.collide(b, b, 3)
    assert torch.equal(a, b)
    batch = pkg.Batch([kw, dict(kw, nx=8, ny=8)])
    hb, ob = batch.empty(0.0), batch.empty()
    batch.view(hb, 0).copy_(h)
    batch.set_step(3)
    batch.step(hb, ob, [w, w])
    got = batch.view(ob, 0)
    assert float((got - a).abs().max()) <= 1e-6 * float(a.abs().max())
