"""The P2G tile at its edges: nodes that only tiny weights reach.

Particles are placed a distance delta (down to 2^-17 of a cell, and zero) above
a cell edge, alone and in clusters, so that some nodes of a chunk's box take
nothing but weights far below one fixed-point unit of the tile, and some
take such weights beside ordinary ones.  Every node's velocity is compared
with the FP64 oracle's normwise (a node whose momentum and mass were resolved
to few units would be off by its whole velocity), and every node's mass
relative to itself: a weight is a product of three quadratics of FP32
offsets that are exact here, so it is good to a few times 2^-24.
"""
import numpy as np
import pytest

from paper_2111_00699_amd import scenes

from .test_gpu_parity import TOL, make_sim, normwise, print_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    return torch


def edge_particles(n, per_cluster, seed):
    """Clusters of `per_cluster` particles in separate places; each axis of each
    particle sits delta above a cell edge (delta = 0 or 2^-17 .. 2^-2 of a cell)
    or, every fourth, anywhere in the cell."""
    k = 0
    out = []
    for cx in range(8, n - 8, 9):
        for cy in range(8, n - 8, 9):
            u = scenes.uniform(seed, 6 * per_cluster, k).reshape(per_cluster, 2, 3)
            k += 1
            delta = np.where(u[:, 0] < 0.05, 0.0, 2.0 ** -np.floor(2 + 16 * u[:, 0]))
            delta = np.where(u[:, 1] < 0.25, u[:, 0], delta)
            cell = np.array([cx, cy, 8 + (k * 5) % (n - 18)]) + np.floor(2 * u[:, 1])
            out.append((cell + 0.5 + delta) / n)
    return np.ascontiguousarray(np.concatenate(out).T.astype(np.float32))


@pytest.mark.parametrize("per_cluster", [1, 3, 40])
@pytest.mark.parametrize("chunk", [64, 256, 512])
@pytest.mark.parametrize("steps", [1, 2])
def test_nodes_reached_by_tiny_weights_only(torch_cuda, oracle, per_cluster, chunk, steps):
    n = 64
    x = edge_particles(n, per_cluster, 90 + per_cluster)
    st = scenes.nontrivial_state(x, seed=41, kind="jelly")
    cfg = dict(n=n, dt=1e-4, bc="separate", bc_cells=3, gravity=(0.0, -9.8, 0.0))
    print_case("tiny_weights", N=x.shape[1], per_cluster=per_cluster, chunk=chunk, steps=steps)
    sim = make_sim(torch_cuda, cfg, chunk=chunk)
    sim.add_particles(scenes.JELLY, st["x"], v=st["v"], C=st["C"], F=st["F"])
    sim.substep(steps)
    assert sim.stats()["p2g_global_particles"] == 0  # every particle took the tile
    gm, gv = (t.cpu().numpy() for t in sim.read_grid())
    sim.close()
    _, om, ov, bad = oracle.substep(cfg, scenes.JELLY, st, steps=steps)
    assert bad == 0
    assert normwise(gm, om) <= TOL
    if steps == 1:  # (later the FP32 positions themselves differ from the oracle's)
        seen = om > 1e-30  # normal FP32 masses with room below
        assert seen.sum() > 0 and om[seen].min() < 1e-14
        assert np.abs(gm[seen] / om[seen] - 1.0).max() <= 1e-5
        # a particle exactly on an edge gives its outer nodes a weight of zero: they stay empty
        assert np.all(gm[om == 0.0] == 0.0)
        vv, oo = gv.reshape(3, -1)[:, seen], ov.reshape(3, -1)[:, seen]
        assert np.abs(vv - oo).max() <= TOL * np.abs(oo).max()
