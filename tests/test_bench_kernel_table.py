"""bench.py's per-launch table of the plain form, from event totals over several steps of several frames:
each kind's bytes are those of the levels it covers, whichever of them share a launch."""
import importlib.util
from pathlib import Path

import pytest

import paper_1810_03988_amd as P
import workloads as wl

spec = importlib.util.spec_from_file_location("bench", Path(__file__).resolve().parents[1] / "bench.py")
bench = importlib.util.module_from_spec(spec)
spec.loader.exec_module(bench)


@pytest.mark.parametrize("passes, middle, top", [(4, 4, True), (3, 2, True), (1, 0, True), (1, 0, False)])
@pytest.mark.parametrize("steps, frames", [(1, 1), (5, 30)])
def test_bytes_of_a_frame(passes, middle, top, steps, frames):
    rig = wl.rig_c2()
    plan = P.Plan(rig.frame_sizes, rig.H, rig.masks(), rig.canvas_w, rig.canvas_h, rig.levels, device="cpu", bind=False)
    n = steps * frames
    timing = {"warp_level0_pass": (1.0 * n, n), "level_pass": (1.0 * n, passes * n), "blend_level0": (1.0 * n, n)}
    if middle:
        timing["blend_middle"] = (1.0 * n, middle * n)
    if top:
        timing["blend_top"] = (1.0 * n, n)
    table = bench.kernel_table(plan, rig, timing, steps, 4)
    assert table.keys() == timing.keys()
    ph = bench.phase_bytes(plan, rig, 4)
    got = sum(r["alg_bytes_per_launch"] * timing[k][1] / n for k, r in table.items())
    assert abs(got - sum(ph.values())) <= passes + middle + 3       # (whole bytes a launch)


@pytest.mark.parametrize("passes, blends", [(5, 6), (3, 4), (1, 1)])
def test_bytes_of_a_batch(passes, blends):
    """Levels 0 .. passes - 1 and 0 .. blends - 1 timed, the last of each with those above it."""
    rig = wl.rig_c2()
    plan = P.Plan(rig.frame_sizes, rig.H, rig.masks(), rig.canvas_w, rig.canvas_h, rig.levels, device="cpu", bind=False)
    timing = {("pyr", k): (2.0, 2) for k in range(passes)} | {("blend", k): (2.0, 2) for k in range(blends)}
    table = bench.batch_kernel_table(plan, rig, timing, 2, 2, 7)
    got = sum(r["alg_bytes_per_launch"] for r in table.values())
    assert got == 7 * sum(bench.phase_bytes(plan, rig, 2).values())
