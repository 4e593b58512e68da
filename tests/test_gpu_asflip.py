"""ASFLIP transfer and the automatic frame step on the GPU against the FP64
oracle (om_substep_asflip, oracle.frame_time_step).

* One and five substeps with ASFLIP (flip 0.95, beta 0 / 1) from the random
  water and jelly states: every particle field within 1e-4, as for APIC;
  positions of the particles whose J' came within 1e-6 of 1 in some
  substep (where FP32 and FP64 may pick different betas) are left out of
  that bar and held to 2e-4.
* flip = 0 leaves the APIC path untouched, bit for bit.
* The fountain partway through a run, with ASFLIP and the automatic step:
  the frame's substep count is the oracle's rule applied to the same FP32
  velocities, and the frame matches the oracle on totals and bounding
  statistics (mass, momentum, bounding box, centre of mass, kinetic energy).
"""
import numpy as np
import pytest

from paper_2111_00699_amd import scenes

from .test_gpu_multistep import compare_totals, totals
from .test_gpu_parity import compare_state, gpu_state, make_sim, normwise, print_case

pytestmark = pytest.mark.gpu

FLIP, BMIN, BMAX = 0.95, 0.0, 1.0


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    return torch


@pytest.mark.parametrize("kind", ["water", "jelly"])
@pytest.mark.parametrize("steps", [1, 5])
def test_asflip_substeps_match_oracle(torch_cuda, oracle, kind, steps):
    mat = scenes.WATER if kind == "water" else scenes.JELLY
    bc = "separate" if kind == "water" else "sticky"
    st = scenes.nontrivial_state(scenes.jelly_cube(0)["x"], seed=5, kind=kind)
    cfg = dict(n=64, dt=1e-4, bc=bc)
    print_case("asflip", kind=kind, steps=steps)
    sim = make_sim(torch_cuda, cfg)
    sim.add_particles(mat, st["x"], v=st["v"], C=st["C"], F=st.get("F"), s=st.get("s"))
    sim.set_transfer(FLIP, BMIN, BMAX)
    sim.substep(steps)
    gs = gpu_state(sim)
    assert sim.stats()["error"] == 0
    sim.close()
    # the oracle one substep at a time, keeping each particle's closest approach of J' to 1:
    # beta is chosen by J' < 1, which FP32 and FP64 may decide differently within rounding
    os_, jgap, bad = dict(st), np.full(st["x"].shape[1], np.inf), 0
    for _ in range(steps):
        J0 = np.asarray(os_.get("s", np.ones(st["x"].shape[1])), np.float64)
        os_, _, _, b = oracle.substep_asflip(cfg, mat, os_, FLIP, BMIN, BMAX)
        bad += b
        G = np.eye(3)[None] + cfg["dt"] * os_["C"].T.reshape(-1, 3, 3)
        J = np.linalg.det(G) * (J0 if kind == "water" else 1.0)
        jgap = np.minimum(jgap, np.abs(J - 1.0))
    assert bad == 0
    near = jgap < 1e-6
    print(f"[asflip] beta decisions within 1e-6 of J' = 1: {near.sum()} of {near.size}", flush=True)
    assert near.mean() < 0.01
    keep = ~near
    errs = compare_state({**gs, "x": gs["x"][:, keep]}, {**os_, "x": os_["x"][:, keep]}, kind, n=cfg["n"],
                         label=f"asflip {kind} x{steps}")
    assert normwise(gs["x"], os_["x"]) <= 2e-4  # every particle, beta flips included
    # the transfer did act: APIC differs from it by far more than the bar
    ap, _, _, _ = oracle.substep(cfg, mat, st, steps=steps)
    assert normwise(os_["v"], ap["v"]) > 1e-2


def test_flip_zero_is_the_apic_path(torch_cuda):
    st = scenes.nontrivial_state(scenes.jelly_cube(0)["x"], seed=5, kind="water")
    cfg = dict(n=64, dt=1e-4, bc="separate")
    out = []
    for flip in (None, 0.0):
        sim = make_sim(torch_cuda, cfg)
        sim.add_particles(scenes.WATER, st["x"], v=st["v"], C=st["C"], s=st["s"])
        if flip is not None:
            sim.set_transfer(flip, BMIN, BMAX)
        sim.substep(3)
        out.append(gpu_state(sim))
        sim.close()
    for k in ("x", "v", "C", "s"):
        assert np.array_equal(out[0][k], out[1][k]), k


def test_fountain_frame_with_asflip_and_automatic_step(torch_cuda, oracle):
    cfg0 = scenes.fountain_config()
    n = cfg0["n"]
    frame = np.float32(scenes.FRAME)
    cfl, dt_max = np.float32(0.3), np.float32(1e-3)
    e = scenes.fountain_emission(30)
    base = scenes.fountain_midrun(limit=143500 - e["x"].shape[1])
    st = {"x": np.concatenate([base["x"], e["x"]], axis=1), "v": np.concatenate([base["v"], e["v"]], axis=1)}
    N = st["x"].shape[1]
    sim = make_sim(torch_cuda, dict(n=n, dt=cfg0["dt"], bc=cfg0["bc"], bc_cells=cfg0["bc_cells"],
                                    gravity=cfg0["gravity"]))
    sim.add_particles(scenes.WATER, base["x"], v=base["v"])
    sim.add_particles(None, e["x"], v=e["v"])
    sim.set_transfer(FLIP, BMIN, BMAX)
    sim.set_auto_dt(float(cfl), float(dt_max))
    sim.frame(float(frame))
    sim.synchronize()
    ss = sim.scene_stats()
    gs = gpu_state(sim)
    assert sim.stats()["error"] == 0
    sim.close()
    # the oracle's rule on the same FP32 velocities (FP32 constants as the library holds them)
    v = st["v"].astype(np.float32)
    vmax = float(np.sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]).max())
    g = tuple(float(np.float32(a)) for a in cfg0["gravity"])
    ns, dt = oracle.frame_time_step(scenes.WATER, n, vmax, g, float(cfl), float(dt_max), float(frame))
    print_case("fountain_asflip_auto_dt", N=N, substeps=ns, dt=dt, gpu_substeps=ss["substeps"], gpu_dt=ss["dt"])
    assert ns < cfg0["substeps_per_frame"] / 2  # the automatic step is much longer than the fixed one
    assert ss["substeps"] == ns
    assert abs(ss["dt"] - dt) <= 1e-6 * dt
    cfg = dict(n=n, dt=dt, bc=cfg0["bc"], bc_cells=cfg0["bc_cells"], gravity=cfg0["gravity"])
    os_, om, _, bad = oracle.substep_asflip(cfg, scenes.WATER, st, FLIP, BMIN, BMAX, steps=ns)
    assert bad == 0
    mp = scenes.WATER["rho"] / n ** 3 / scenes.WATER["ppc"]
    g_, o_ = totals(gs, mp), totals(os_, mp)
    scale = max(o_["mv"].max(), g_["mv"].max())
    print(f"[momentum] gpu={g_['P']} oracle={o_['P']} scale={scale:.3e}", flush=True)
    assert np.abs(g_["P"] - o_["P"]).max() <= 1e-2 * scale
    compare_totals(g_, o_, n, "fountain asflip auto-dt")


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("chunk", [64, 256, 512])
def test_another_scenes_map_leaves_asflip_water_bit_for_bit(torch_cuda, mode, chunk):
    """An ASFLIP scene's sums are rounded the same whatever map another scene of its context takes: the
    water of a water and snow context with the learned (1) or closed-form (2) snow map against the same
    with the exact map.  (Its scatter is exact, so nothing depends on the order of the adds.)"""
    from paper_2111_00699_amd import mpm

    water = scenes.nontrivial_state(scenes.jelly_cube(0)["x"], seed=5, kind="water")
    snow = scenes.nontrivial_state(scenes.jelly_cube(0)["x"], seed=6, kind="snow")
    print_case("asflip_beside_map", mode=mode, chunk=chunk)
    sur = mpm.Surrogate()
    sur.set(scenes.mlp_init(4), np.concatenate([np.zeros(12), np.ones(12)] * 2).astype(np.float32))
    out = []
    for m in (0, mode):
        sim = mpm.Sim(64, 1e-4, scenes=[dict(n=64, dt=1e-4, bc="separate")] * 2, chunk=chunk)
        sim.add_particles(scenes.WATER, water["x"], v=water["v"], C=water["C"], s=water["s"], scene=0)
        sim.add_particles(scenes.SNOW, snow["x"], v=snow["v"], C=snow["C"], F=snow["F"], s=snow["s"], scene=1)
        sim.set_transfer(FLIP, BMIN, BMAX, scene=0)
        if m:
            sim.use_surrogate(m, sur, tol=1e-2, dt_ref=1e-4, scene=1)
        sim.substep(3)
        stats = sim.stats()
        assert stats["p2g_global_particles"] == 0
        assert (stats["surrogate_particles"] + stats["surrogate_fallbacks"] > 0) == (m != 0)
        out.append({k: t.cpu().numpy() for k, t in sim.read_particles(scene=0).items()})
        sim.close()
    for k in ("x", "v", "C", "s"):
        assert np.array_equal(out[0][k], out[1][k]), k
    sur.close()
