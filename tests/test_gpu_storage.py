"""Storage order in and out: a state that is only sorted comes back bit for bit.

A rebuild sorts and permutes the stored particles and a read copies them back
to insertion order.  Particles at rest, without stress or gravity, also pass
their substep unchanged (every sum is an exact zero), so x, F and s come back
exactly at every size: around the sort's tiles (2048 keys), the size where
it changes its tiles and its histogram (262144), and the size from which a
read sorts each group of 256 by insertion id (131072).  Before a substep every
field does.
"""
import numpy as np
import pytest

from paper_2111_00699_amd import scenes

from .test_gpu_parity import gpu_state, make_sim, print_case

pytestmark = pytest.mark.gpu
FIELDS = ("x", "v", "C", "F", "s")


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    return torch


REST = dict(scenes.JELLY, E=0.0)


def cloud(N, seed, moving=False):
    x = scenes.uniform(seed, 3 * N, 0, 0.05, 0.95).reshape(3, -1).astype(np.float32)
    st = {k: np.asarray(a, np.float32) for k, a in scenes.nontrivial_state(x, seed=seed + 1, kind="snow").items()}
    if not moving:
        st["v"], st["C"] = np.zeros_like(st["v"]), np.zeros_like(st["C"])
    return st


def add(sim, st, scene=0, mat=REST):
    sim.add_particles(mat, st["x"], v=st["v"], C=st["C"], F=st["F"], s=st["s"], scene=scene)


def assert_same(got, st):
    for k in FIELDS:
        assert np.array_equal(np.asarray(got[k]).reshape(-1), st[k].reshape(-1)), k


@pytest.mark.parametrize("N", [1, 255, 257, 131071, 131072, 131073])
def test_state_reads_back_before_a_substep(torch_cuda, N):
    print_case("inserted_state", N=N)
    st = cloud(N, 300 + N % 1000, moving=True)
    sim = make_sim(torch_cuda, dict(n=64, dt=1e-5))
    add(sim, st)
    assert_same(gpu_state(sim), st)
    sim.close()


@pytest.mark.parametrize("chunk", [0, 64, 512])
@pytest.mark.parametrize("N", [1, 255, 2047, 2048, 2049, 131071, 131073, 262143, 262144, 262145])
def test_sorted_state_reads_back_exactly(torch_cuda, oracle, N, chunk):
    print_case("sorted_state", N=N, chunk=chunk)
    st = cloud(N, 300 + N % 1000)
    sim = make_sim(torch_cuda, dict(n=64, dt=1e-5, gravity=(0, 0, 0)), chunk=chunk)
    add(sim, st)
    for _ in range(2):  # the second sorts the storage order of the first
        sim.rebuild()
        sim.substep(1)
        assert_same(gpu_state(sim), st)
    keys, _ = sim.read_binning()
    assert np.array_equal(keys, oracle.bin_particles(st["x"], 64)["sorted"])
    sim.close()


@pytest.mark.parametrize("sizes", [(1, 700, 3), (5000, 131072, 300)])
def test_scene_reads_cover_their_storage(torch_cuda, sizes):
    from paper_2111_00699_amd import mpm

    print_case("scene_reads", sizes=sizes)
    # (storage order is by rank: the last scene has the smallest dt)
    descs = [dict(n=64, dt=(3 - k) * 1e-5, bc="sticky") for k in range(3)]
    sim = mpm.Sim(64, 1e-5, scenes=descs, gravity=(0, 0, 0))
    sts = [cloud(N, 400 + k) for k, N in enumerate(sizes)]
    for k, st in enumerate(sts):
        add(sim, st, scene=k)

    def check():
        for k, st in enumerate(sts):
            assert_same({f: t.cpu().numpy() for f, t in sim.read_particles(scene=k).items()}, st)

    check()  # insertion order
    sim.substep(1)
    check()  # sorted
    extra = cloud(257, 500)
    add(sim, extra, scene=0, mat=None)
    sts[0] = {f: np.concatenate([sts[0][f].reshape(-1, sizes[0]), extra[f].reshape(-1, 257)], axis=1) for f in FIELDS}
    check()  # appended behind the sorted ones
    sim.substep(1)
    check()
    sim.close()


@pytest.mark.parametrize("sizes", [(131072, 131072), (131072, 131073), (300, 131072), (131071, 131073), (140000, 500000)])
def test_scene_reads_before_the_first_rebuild(torch_cuda, sizes):
    """Reads out of storage that holds other scenes too, at the sizes where the sort of a group begins (the
    scene's particles, and their share of the positions)."""
    print_case("unsorted_scene_reads", sizes=sizes)
    sim = make_sim(torch_cuda, dict(n=64, dt=1e-5), num_scenes=2)
    sts = [cloud(N, 420 + k, moving=True) for k, N in enumerate(sizes)]
    for k, st in enumerate(sts):
        add(sim, st, scene=k)
    for k, st in enumerate(sts):
        assert_same({f: t.cpu().numpy() for f, t in sim.read_particles(scene=k).items()}, st)
    sim.close()


def test_read_of_a_small_scene_costs_a_scan(torch_cuda):
    """A scene of 1,000 particles among 16M that no rebuild has sorted: its read looks at one word per
    position, 4 bytes against the 104 that the read of the 16M moves each way, and took 0.06 of that read's
    time (0.27 when every group was sorted for it)."""
    import time

    torch, big = torch_cuda, 1 << 24
    print_case("small_scene_read", big=big)
    sim = make_sim(torch, dict(n=128, dt=1e-5), num_scenes=2, capacity=2 * big + 4096)
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    for k, N in enumerate((big, 1000)):
        sim.add_particles(scenes.WATER, 0.05 + 0.9 * torch.rand((3, N), device="cuda", generator=g), scene=k)
    best = []
    for k in range(2):
        times = []
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            sim.read_particles(scene=k)
            times.append(time.perf_counter() - t)
        best.append(min(times))
    sim.close()
    print(f"[time] read of {big} {best[0] * 1e6:.0f} us, of 1000 {best[1] * 1e6:.0f} us", flush=True)
    assert best[1] <= 0.15 * best[0]


@pytest.mark.parametrize("N", [8192 * 2048, 8192 * 2048 + 1])
def test_blocks_on_both_sides_of_the_scans_line(torch_cuda, N):
    """From 8193 tiles of 2048 particles on, the block scan's totals are scanned by a launch of their own:
    the blocks are those of the sorted codes, and the state comes back bit for bit."""
    from paper_2111_00699_amd import mpm

    torch = torch_cuda
    print_case("scan_line_particles", N=N)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = 0.05 + 0.9 * torch.rand((3, N), device="cuda", generator=g)
    sim = make_sim(torch, dict(n=256, dt=1e-5, gravity=(0, 0, 0)), capacity=N, flags=mpm.FLAG_ALLOC_EXACT)
    sim.add_particles(REST, x)
    sim.substep(1)
    assert torch.equal(sim.read_particles()["x"], x)
    keys, perm = sim.read_binning()
    blocks = sim.read_blocks()
    stats = sim.stats()
    sim.close()
    assert np.all(keys[1:] >= keys[:-1])
    start = np.flatnonzero(np.concatenate([[True], keys[1:] >> 6 != keys[:-1] >> 6]))
    assert np.array_equal(blocks["gstart"], start)
    assert np.array_equal(blocks["gcode"], keys[start] >> 6)
    assert np.array_equal(blocks["gcount"], np.diff(np.concatenate([start, [N]])))
    assert np.array_equal(np.bincount(perm, minlength=N), np.ones(N, np.int64))
    # (the chunks follow from the blocks: consecutive ones of a 2x2x1 slab, packed up to 256 particles)
    assert stats["chunks"] >= N // 256 and stats["p2g_global_particles"] == 0


def test_chunk_and_active_block_scans_above_the_line(torch_cuda, oracle):
    """Eight scenes of 512^3 cells hold 17.6M blocks (8,582 tiles of 2048), and 2.2M particles may begin as
    many chunks (8,594 tiles of 256): both scans take the launch for the totals."""
    from paper_2111_00699_amd import mpm

    per = 275000
    print_case("scan_line_blocks", per=per)
    sim = mpm.Sim(512, 1e-5, num_scenes=8, gravity=(0, 0, 0), capacity=8 * per, flags=mpm.FLAG_ALLOC_EXACT)
    xs = [scenes.uniform(510 + k, 3 * per, 0, 0.05, 0.95).reshape(3, -1).astype(np.float32) for k in range(8)]
    for k, x in enumerate(xs):
        sim.add_particles(REST, x, scene=k)
    sim.substep(1)
    for k, x in enumerate(xs):
        assert np.array_equal(sim.read_particles(scene=k)["x"].cpu().numpy(), x), k
    for k in (0, 5, 7):
        keys, perm = sim.read_binning(scene=k)
        blocks = sim.read_blocks(scene=k)
        ref = oracle.bin_particles(xs[k], 512)
        for got, want in ((keys, "sorted"), (perm, "perm"), (blocks["gcode"], "gblock"), (blocks["gstart"], "gstart"),
                          (blocks["gcount"], "gcount"), (blocks["active"], "pblock")):
            assert np.array_equal(got, ref[want]), (k, want)
    sim.close()
