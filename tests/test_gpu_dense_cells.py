"""Many particles in few cells: chunks whose tile is kept in several copies.

A chunk with at least 8 particles per cell of its box scatters into 2 to 8 or
16 copies of its tile, as many as its particles fill and the tile's memory
holds, and sums them when it stores the tile.  The sums are whole numbers, so
the bars are those of any other substep: the grid and the state against the
FP64 oracle's, normwise, at particle counts around the thresholds and far
above them, in one cell and in eight.
"""
import numpy as np
import pytest

from paper_2111_00699_amd import scenes

from .test_gpu_parity import TOL, gpu_state, make_sim, normwise, print_case

pytestmark = pytest.mark.gpu
SITES = [(9, 9, 9), (40, 12, 20), (21, 33, 50), (50, 50, 14)]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    return torch


def clusters(n, per, span, seed):
    out = []
    for k, site in enumerate(SITES):
        u = scenes.uniform(seed, 3 * per, k, 0.02, 0.98).reshape(per, 3)
        out.append((np.array(site) + 0.5 + span * u) / n)
    return np.ascontiguousarray(np.concatenate(out).T.astype(np.float32))


@pytest.mark.parametrize("flip", [0.0, 0.9])
@pytest.mark.parametrize("per,span,chunk", [(7, 1, 0), (8, 1, 0), (15, 1, 64), (64, 1, 64), (65, 2, 64), (256, 1, 0), (255, 2, 0),
                                            (511, 1, 512), (3001, 1, 0), (3000, 2, 512)])
def test_crowded_cells_match_the_oracle(torch_cuda, oracle, per, span, chunk, flip):
    n = 64
    st = scenes.nontrivial_state(clusters(n, per, span, 700 + per), seed=71, kind="water")
    cfg = dict(n=n, dt=1e-5, bc="separate", bc_cells=3, gravity=(0.0, -9.8, 0.0))
    print_case("crowded_cells", per=per, span=span, chunk=chunk, flip=flip)
    for steps in (1, 2):
        sim = make_sim(torch_cuda, cfg, chunk=chunk)
        sim.add_particles(scenes.WATER, st["x"], v=st["v"], C=st["C"], F=st.get("F"), s=st["s"])
        if flip:
            sim.set_transfer(flip, 0.0, 1.0)
        sim.substep(steps)
        gs = gpu_state(sim)
        gm, gv = (t.cpu().numpy() for t in sim.read_grid())
        assert sim.stats()["p2g_global_particles"] == 0
        sim.close()
        if flip:
            os_, om = st, None
            for _ in range(steps):
                os_, om, ov, bad = oracle.substep_asflip(cfg, scenes.WATER, os_, flip, 0.0, 1.0)
                assert bad == 0
        else:
            os_, om, ov, bad = oracle.substep(cfg, scenes.WATER, st, steps=steps)
            assert bad == 0
        assert normwise(gm, om) <= TOL
        assert normwise(gv, ov) <= TOL
        for k in ("x", "v"):
            assert normwise(gs[k], os_[k]) <= TOL, k
