"""Workgroup sizes of the collision: both sides of every line of the rule (one,
two and three cells per CU, light and heavy pair loops, shared, drawn and
continuous pairs), each against the FP64 oracle on cells spread over the grid.
Bar of the collision tests: 1e-5 of each cell's largest value.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# threads of the shared-record kernel expected where a CU gets the cells of
# the case (MI355X: 256 CUs)
CASES = [
    dict(nx=16, ny=16, n_pairs=511, block=256),    # one cell a CU, light
    dict(nx=16, ny=16, n_pairs=512, block=1024),   # one cell a CU
    dict(nx=257, ny=1, n_pairs=512, block=256),    # two cells, three workgroups fit
    dict(nx=257, ny=1, n_pairs=512, nv=(16, 16, 16), vmax=5.0, block=512),   # two cells, two fit
    dict(nx=257, ny=1, n_pairs=511, nv=(16, 16, 16), vmax=5.0, block=256),   # ... light
    dict(nx=19, ny=27, n_pairs=767, block=256),    # three cells, light draws
    dict(nx=19, ny=27, n_pairs=768, block=256),
    dict(nx=24, ny=16, n_pairs=767, block=256),    # two cells, light draws
    dict(nx=24, ny=16, n_pairs=768, block=256),
]


@pytest.mark.parametrize("pairs", ["shared", "own", "continuous"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_collide_block_rule(oracle_mod, case, pairs):
    import torch

    import paper_1005_5405_amd as pkg

    kw = dict(dict(nv=(8, 6, 5), vmax=3.0), **CASES[case])
    block = kw.pop("block")
    kw = dict(kw, delta=10.0, eps=0.1, bc=1, mix16=4, sample_group=0 if pairs == "shared" else 1,
              flags=4 if pairs == "continuous" else 0)
    print("[gpu-case] collision blocks", kw, flush=True)
    g, o = pkg.Boltz(**kw), oracle_mod.Oracle(**kw)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert g.collide_block == block
    h = (0.2 * np.random.default_rng(case).standard_normal((g.ncells, g.nv))).astype(np.float32)
    out = g.empty()
    g.collide(torch.from_numpy(h).cuda(), out, 3)
    got = out.cpu().numpy().reshape(-1, g.nv)
    cells = np.unique(np.linspace(0, g.ncells - 1, 9).astype(np.int64))
    ref = o.collide_cells(h[cells].astype(np.float64), 3, cells)
    assert (np.abs(got[cells] - ref).max(1) <= 1e-5 * np.abs(ref).max(1)).all()
    assert g.read_status() == 0
