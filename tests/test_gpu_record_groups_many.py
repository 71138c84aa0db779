"""Grouped shared records (rearranged by first node) with several sample groups,
each group's cells against the FP64 oracle, in the collision, the step's face
launches and a batch; and with increments so large that terms leave the
fixed-point window.  Bars: 1e-5 of each cell's largest value (FP32 state and
coefficients); for the large increments 1e-5 of each node's sum of absolute
terms (a few ulps a term, FP32 sums of the terms outside the window).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# record-cells >= 6e7 and >= 512 cells a group select the grouped form
GROUPS = [
    dict(nx=64, ny=64, nv=(8, 6, 4), vmax=3.0, n_pairs=20481, sample_group=2048),        # five blocks + one record
    dict(nx=60, ny=35, nv=(5, 7, 4), vmax=3.0, n_pairs=30001, sample_group=700),         # three groups
    dict(nx=64, ny=32, nv=(22, 24, 24), vmax=5.0, n_pairs=40001, sample_group=1024),     # partial-tile layout
]


def _state(o, seed):
    return (0.2 * np.random.default_rng(seed).standard_normal((o.ny, o.nx, o.nv))).astype(np.float32)


@pytest.mark.parametrize("case", range(len(GROUPS)))
def test_collide_each_group(oracle_mod, case):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(GROUPS[case], delta=10.0, eps=0.1, bc=1, mix16=4)
    print("[gpu-case] grouped records, each sample group", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    h = _state(g, case)
    out = g.empty()
    g.collide(torch.from_numpy(h).cuda(), out, 7)
    got = out.cpu().numpy().reshape(-1, g.nv)
    per = kw["sample_group"]
    cells = np.array([c + d for c in range(0, g.ncells, per) for d in (0, 1, per // 2, per - 1)])
    assert len(set(cells // per)) == (g.ncells + per - 1) // per > 1
    ref = o.collide_cells(h.reshape(-1, g.nv)[cells].astype(np.float64), 7, cells)
    err = np.abs(got[cells] - ref).max(1)
    assert (err <= 1e-5 * np.abs(ref).max(1)).all(), err / np.abs(ref).max(1)
    assert g.read_status() == 0


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("case", range(2))
def test_step_and_batch_each_group(case, order):
    """Records drawn and grouped in the face launches, and by the batch: equal
    to streaming and colliding one after the other, in every sample group."""
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(GROUPS[case], delta=10.0, eps=0.1, mix16=4, order=order)
    g = pkg.Boltz(**kw)
    w = pkg.Walls(lid_u=0.1, tau_left=1.02)
    h = torch.from_numpy(_state(g, 5 + case)).cuda()
    a, b = g.empty(), g.empty()
    g.step(h, a, w, 3)
    g.stream(h, b, w)
    g.collide(b, b, 3)
    assert torch.equal(a, b)
    batch = pkg.Batch([kw, dict(kw, nx=8, ny=8), dict(GROUPS[1 - case], delta=5.0, eps=0.1, mix16=4, order=order)])
    hb, ob = batch.empty(0.0), batch.empty()
    batch.view(hb, 0).copy_(h)
    batch.set_step(3)
    batch.step(hb, ob, [w, w, w])
    # another block size than the single problem's: the order of the FP64 sums only
    d = (batch.view(ob, 0) - a).abs().reshape(g.ncells, -1).max(1).values
    assert bool((d <= 1e-6 * a.abs().reshape(g.ncells, -1).max(1).values).all())


@pytest.mark.parametrize("kw", [
    dict(nx=64, ny=32, nv=(6, 6, 8), vmax=3.0, n_pairs=32768, delta=1.0e11),
    dict(nx=40, ny=40, nv=(22, 24, 24), vmax=5.0, n_pairs=40001, delta=1.0e10),
])
def test_collide_grouped_beyond_window(oracle_mod, kw):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(kw, sample_group=0, eps=0.1, bc=1, mix16=4, dt=0.002)
    print("[gpu-case] grouped records beyond the window", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    h = _state(g, 9)
    out = g.empty()
    g.collide(torch.from_numpy(h).cuda(), out, 7, correction=False)
    got = out.cpu().numpy().reshape(-1, g.nv)
    cells = np.array([0, 1, g.ncells // 2, g.ncells - 1])
    hc = h.reshape(-1, g.nv)[cells].astype(np.float64)
    ref = o.collide_cells(hc, 7, cells, correction=False)
    idx, q = o.debug_pairs(0, 7, 0, kw["n_pairs"])
    a, b, s, t = idx[idx[:, 2] >= 0].T
    q = q[idx[:, 2] >= 0]
    w = o.node_weights().reshape(-1)[: o.nv]
    for k in range(len(cells)):
        mag = np.abs(hc[k])[a] + np.abs(hc[k])[b] + 0.1 * np.abs(hc[k][a] * hc[k][b])
        total = np.abs(hc[k]).copy()
        for j in (s, t, a, b):
            np.add.at(total, j, q / w[j] * mag)
            big = q / w[j] * np.abs(hc[k][a] + hc[k][b] + 0.1 * hc[k][a] * hc[k][b]) > 2.0 ** 18
            assert 0.001 < big.mean() < 0.9
        err = np.abs(got[cells[k]] - ref[k])
        assert (err <= 1e-5 * total).all(), (err / total).max()
    assert g.read_status() == 0


@pytest.mark.parametrize("kw", [
    dict(nx=24, ny=20, nv=(20, 20, 20), vmax=5.0, n_pairs=20833),     # below 1e7 record-cells: in order
    dict(nx=24, ny=20, nv=(20, 20, 20), vmax=5.0, n_pairs=20834),     # dealt with the y faces, in order alone
    dict(nx=64, ny=40, nv=(6, 6, 8), vmax=3.0, n_pairs=9765),         # small tile below 2.5e7: in order
    dict(nx=64, ny=40, nv=(6, 6, 8), vmax=3.0, n_pairs=9766),         # grouped
])
def test_step_at_the_lines_of_the_record_rule(oracle_mod, kw):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(kw, delta=10.0, eps=0.1, mix16=4, sample_group=0)
    print("[gpu-case] record rule", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    w = pkg.Walls(lid_u=0.1)
    h = torch.from_numpy(_state(g, 3)).cuda()
    a, b, hs = g.empty(), g.empty(), g.empty()
    g.step(h, a, w, 3)
    g.stream(h, hs, w)
    g.collide(hs, b, 3)
    assert torch.equal(a, b)
    cells = np.array([0, 7, g.ncells // 2, g.ncells - 1])
    ref = o.collide_cells(hs.cpu().numpy().reshape(-1, g.nv)[cells].astype(np.float64), 3, cells)
    err = np.abs(a.cpu().numpy().reshape(-1, g.nv)[cells] - ref).max(1)
    assert (err <= 1e-5 * np.abs(ref).max(1)).all()
    assert g.read_status() == 0
