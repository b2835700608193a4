"""GPU tests of the collision kernel's bounds: steps at which the boxes of two
groups of trajectories lie apart are not tested, with the results of testing
every step. Scenes at the edges of the groups (8 trajectories a box, 32 a
block), of the step windows (64, 128) and of what a box can separate, against
the oracle and against the same kernel laid out without boxes (a context whose
budget holds the workspace only without them), which tests every step."""
import math

import numpy as np
import pytest

import oracle
from paper_2005_06773_amd import scenegen as sg
from tests import parity
from tests.random_scenes import random_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mhc():
    from paper_2005_06773_amd import mhc as m
    return m


@pytest.fixture(scope="module")
def ctx(mhc):
    c = mhc.mhc_create(0)
    yield c
    mhc.mhc_destroy(c)


def _without_boxes(mhc, scene):
    """The scene's results from a context that has no room for the boxes."""
    cs = mhc.CScene(scene)
    boxes = sum((cs.H * ((t + 7) // 8) * 16 + 255) // 256 * 256 for t in cs.T)
    c = mhc.mhc_create(0, mhc.mhc_query_sizes(cs)["device_bytes"] - boxes)
    try:
        return mhc.mhc_evaluate(c, cs)
    finally:
        mhc.mhc_destroy(c)


def _vehicle(rng, n_u, n_w, spread):
    return sg.SceneObject(sg.VEHICLE, float(rng.uniform(-spread, spread)), float(rng.uniform(-spread, spread)),
                          float(rng.uniform(0, 2 * math.pi)), float(rng.uniform(0, 14)), 4.4, 1.8, 0.0,
                          sg.accel_grid(n_u), sg.yaw_grid(n_w), None)


def _pedestrian(rng, n_u, n_w, spread):
    return sg.SceneObject(sg.PEDESTRIAN, float(rng.uniform(-spread, spread)), float(rng.uniform(-spread, spread)),
                          float(rng.uniform(0, 2 * math.pi)), 1.0, 0.0, 0.0, 0.35, sg.ped_speed_grid(n_u),
                          sg.ped_heading_grid(n_w), None)


@pytest.mark.parametrize("grids,horizon", [
    (((1, 1), (7, 1), (8, 1), (3, 3)), 1),
    (((31, 1), (4, 8), (11, 3), (2, 2)), 63),
    (((5, 13), (8, 8), (1, 33), (16, 4)), 64),
    (((9, 7), (3, 11), (6, 43), (1, 2)), 65),
    (((17, 15), (2, 16), (13, 5), (32, 1)), 128),
    (((6, 6), (7, 9), (4, 4), (10, 2)), 129),
    (((3, 5), (5, 3), (2, 9), (9, 2)), 257),
])
def test_group_and_window_edges(mhc, ctx, grids, horizon):
    rng = np.random.default_rng(horizon)
    objs = [_vehicle(rng, *g, 14.0) for g in grids[:2]] + [_pedestrian(rng, *g, 14.0) for g in grids[2:]]
    s = sg.Scene(objs, horizon, 4.0 / max(horizon, 20))
    got = mhc.mhc_evaluate(ctx, s)
    parity.check(s, got, oracle.evaluate(s, threads=8), f"grids {grids} H {horizon}")
    parity.same_results(got, _without_boxes(mhc, s), f"grids {grids} H {horizon}, every step tested")


def test_random_scenes_equal_testing_every_step(mhc, ctx):
    """Every scene option: classes, outlines, motion models, pair and overlap
    modes, readings, the risk over time."""
    for k in range(0, 120, 3):
        s = random_scene(k)
        parity.same_results(mhc.mhc_evaluate(ctx, s), _without_boxes(mhc, s), f"random scene {k}")


@pytest.mark.parametrize("gap", [0.0, 1e-5, 1e-3, 5e-3])
@pytest.mark.parametrize("shift", [0.0, 3.0e4, 1.0e9])
def test_shapes_that_nearly_touch(mhc, ctx, gap, shift):
    """Parallel rectangles, and a circle, `gap` apart along x, near the origin
    and far out, where the rounding of the tests exceeds any gap: the bounds
    may only decide what the tests decide."""
    a = sg.SceneObject(sg.VEHICLE, 0.0, 0.0, 0.0, 0.0, 4.0, 2.0, 0.0, np.zeros(3), np.array([0.0, 1e-7, 2e-7]), None)
    b = sg.SceneObject(sg.VEHICLE, 4.0 + gap, 0.3, 0.0, 0.0, 4.0, 2.0, 0.0, np.zeros(3), np.zeros(3), None)
    c = sg.SceneObject(sg.PEDESTRIAN, -2.5 - gap, 0.1, 0.0, 0.0, 0.0, 0.0, 0.5, np.zeros(2), np.zeros(4), None)
    far = sg.SceneObject(sg.PEDESTRIAN, shift, shift, 0.0, 0.0, 0.0, 0.0, 0.5, np.zeros(1), np.zeros(1), None)
    s = sg.Scene([a, b, c, far], 5, 0.1)
    parity.same_results(mhc.mhc_evaluate(ctx, s), _without_boxes(mhc, s), f"gap {gap} shift {shift}")


def test_poses_that_overflow_are_tested(mhc, ctx):
    """Speeds and headings whose poses leave FP32 or are not finite: a box
    around them separates nothing, so the results stay those of the tests."""
    rng = np.random.default_rng(3)
    objs = [_vehicle(rng, 3, 3, 5.0), _vehicle(rng, 2, 5, 5.0), _pedestrian(rng, 3, 4, 5.0)]
    objs[0].speed = 1e30
    objs[1].u = np.array([0.0, 1e300])
    objs[1].w = np.array([-0.4, 0.0, 0.3, 1e200, 1e308])
    objs[2].u = np.array([0.0, 1.0, 1e25])
    s = sg.Scene(objs, 12, 0.5)
    parity.same_results(mhc.mhc_evaluate(ctx, s), _without_boxes(mhc, s), "overflowing poses")


def test_first_hits_of_split_stages_and_odd_addresses(mhc, ctx):
    """The collision stage writes every first-hit entry of the buffer it is
    given, also when the trajectory stage ran without that buffer, and at
    2-byte addresses."""
    import torch
    s = sg.eleven_object_scene(3)
    ref = mhc.mhc_evaluate(ctx, s)["first_hit"]
    plan = mhc.mhc_plan_create(ctx, s)
    n = len(ref)
    for shift in (0, 1, 3, 7):
        buf = torch.full((n + 16,), 77, dtype=torch.int16, device="cuda")
        out, res = mhc.device_result(plan.cs, first_hit=False)
        res.first_hit = buf.data_ptr() + 2 * shift
        mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_TRAJ)
        mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_COLLIDE, res)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[shift:shift + n], ref), shift
        assert (got[:shift] == 77).all() and (got[shift + n:] == 77).all(), shift
        buf.fill_(77)
        mhc.mhc_plan_execute(plan, res)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert np.array_equal(got[shift:shift + n], ref), shift
        assert (got[:shift] == 77).all() and (got[shift + n:] == 77).all(), shift
    plan.close()


def test_repeated_evaluations_are_identical(mhc, ctx):
    """The tests of a workgroup's blocks are all in before its results are:
    small and mixed scenes, over and over, give the same bytes each time."""
    scenes = [mhc.CScene(s) for s in sg.batch_scenes(7, 48)]
    first = [mhc.mhc_evaluate(ctx, c) for c in scenes]
    for _ in range(15):
        for k, c in enumerate(scenes):
            got = mhc.mhc_evaluate(ctx, c)
            for f in ("first_hit", "q", "traj_crit", "object_crit"):
                assert got[f].tobytes() == first[k][f].tobytes(), (k, f)
