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


def plane_particles(n, count, seed, others):
    """Sites of `count` particles in one cell, each in a chunk of its own: all of a site's particles sit
    the same 2^-15 .. 2^-19 of a cell above a cell edge along one axis (exact in FP32: below cell 16) and
    anywhere in the cell along the other two.  The first `others` of them sit farther from the edge, 2^-10
    .. 2^-14, so that the site's outer nodes hold a few larger weights beside the many."""
    out = []
    for a in range(3):
        for k in range(5):
            u = scenes.uniform(seed, 3 * count, 5 * a + k, 0.1, 0.9).reshape(count, 3)
            u[:, a] = 2.0 ** -(15 + k)
            u[:others, a] = 2.0 ** -(10 + (3 * k + np.arange(others)) % 5)
            site = np.zeros(3)
            site[[a, (a + 1) % 3, (a + 2) % 3]] = 10, 14 + 9 * k, 40
            out.append((site + 0.5 + u) / n)
    x = np.ascontiguousarray(np.concatenate(out).T.astype(np.float32))
    assert all(np.any(np.float64(x[a]) * n == 10.5 + 2.0 ** -19) for a in range(3))
    return x


# A plane's outer nodes collect many equal weights, each far below 2^-32, to any sum.  Bars, all of FP32
# roundings (2^-24 = u): a weight is a product of three quadratics of exact offsets (at most 4 u each and
# 2 u for the products), a tile's sum is stored in FP32 and the grid update adds at most 8 tiles (9 u more):
# 23 u, so 32 u of a node's own mass.  A velocity's numerator sums m = q + Ad o of nine FP32 terms, each up to
# the chunk's largest S (per mass): 9 u S; the weights' errors weigh the particles anew, at most 2 * 14 u S;
# storing and dividing take 9 u S: 46 u, so 64 u of S, which is far above the nodes' own velocities here.
@pytest.mark.parametrize("count,chunk", [(64, 64), (128, 256), (256, 256), (512, 512), (512, 256)])
@pytest.mark.parametrize("moving", [True, False])
@pytest.mark.parametrize("others", [0, 3])
def test_nodes_of_many_equal_tiny_weights(torch_cuda, oracle, count, chunk, moving, others):
    n, u = 64, 2.0 ** -24
    x = plane_particles(n, count, 900 + count, others)
    N = x.shape[1]
    st = dict(x=x, v=np.zeros((3, N), np.float32), C=np.zeros((9, N), np.float32),
              F=np.repeat(np.eye(3, dtype=np.float32).reshape(9, 1), N, axis=1))
    if moving:
        st["v"] = scenes.uniform(17, 3 * N, 0, -1.0, 1.0).reshape(3, N).astype(np.float32)
        st["C"] = scenes.uniform(17, 9 * N, 1, -400.0, 400.0).reshape(9, N).astype(np.float32)
    # no stress (E = 0) and no gravity; the second substep of particles at rest is the fused kernel's
    steps = 1 if moving else 2
    mat = dict(scenes.JELLY, E=0.0)
    cfg = dict(n=n, dt=1e-5, bc="separate", bc_cells=3, gravity=(0.0, 0.0, 0.0))
    print_case("tiny_weight_planes", N=N, count=count, chunk=chunk, moving=moving, others=others)
    sim = make_sim(torch_cuda, cfg, chunk=chunk)
    sim.add_particles(mat, st["x"], v=st["v"], C=st["C"], F=st["F"])
    sim.substep(steps)
    assert sim.stats()["p2g_global_particles"] == 0
    gm, gv = (t.cpu().numpy() for t in sim.read_grid())
    sim.close()
    _, om, ov, bad = oracle.substep(cfg, mat, st, steps=1)
    assert bad == 0
    seen = om > 0.0
    light = seen & (om < 2.0 ** -20 * mat["rho"] / mat["ppc"] / n ** 3)
    assert light.sum() >= 15 * 9  # every plane's nine outer nodes
    em = np.abs(gm[seen] / om[seen] - 1.0).max()
    print(f"[errs] mass {em / u:.1f} u", flush=True)
    assert em <= 32 * u
    if moving:
        f = np.float64(x) * n - np.floor(np.float64(x) * n - 0.5)
        C = np.float64(st["C"]).reshape(3, 3, N) / n
        S = (np.abs(st["v"] - np.einsum("abp,bp->ap", C, f)) + 2 * np.abs(C).sum(axis=1)).max()
        ev = np.abs(gv.reshape(3, -1)[:, seen] - ov.reshape(3, -1)[:, seen]).max()
        print(f"[errs] velocity {ev / (u * S):.1f} u S, S {S:.1f}, largest light |v| "
              f"{np.abs(ov.reshape(3, -1)[:, light]).max():.2f}", flush=True)
        assert ev <= 64 * u * S
    else:
        assert np.all(gv == 0.0)
