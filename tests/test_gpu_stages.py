"""GPU tests of what the separate stages of a plan write."""
import numpy as np
import pytest

from paper_2005_06773_amd import scenegen as sg

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


@pytest.mark.parametrize("stages", [1, 4, 5])     # trajectories, risk, both
@pytest.mark.parametrize("seed,n", [(3, 11), (5, 2)])
def test_stages_without_collisions_leave_the_first_hits(mhc, ctx, stages, seed, n):
    """Only the collision stage writes first hits: the trajectory stage of the
    next frame may run while the last frame's are still to be read, from the
    caller's buffer or from the plan's own."""
    import torch
    s = sg.eleven_object_scene(seed)
    s.objects = s.objects[:n]
    for o in s.objects:
        o.x *= 0.3 if n > 2 else 0.0
        o.y *= 0.3 if n > 2 else 0.0
    want = mhc.mhc_evaluate(ctx, s)["first_hit"]
    assert (want >= 0).any()
    plan = mhc.mhc_plan_create(ctx, s)
    out, res = mhc.device_result(plan.cs)
    mhc.mhc_plan_execute(plan, res)
    mhc.mhc_plan_execute_stages(plan, stages, res)
    torch.cuda.synchronize()
    assert np.array_equal(out["first_hit"].cpu().numpy(), want)
    mhc.mhc_plan_execute(plan)
    mhc.mhc_plan_execute_stages(plan, stages)
    assert np.array_equal(mhc.mhc_plan_download(plan)["first_hit"], want)
    # a trajectory stage and a collision stage apart write what one call does
    mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_TRAJ, res)
    out["first_hit"].fill_(-2)
    mhc.mhc_plan_execute_stages(plan, mhc.MHC_STAGE_COLLIDE, res)
    torch.cuda.synchronize()
    assert np.array_equal(out["first_hit"].cpu().numpy(), want)
    plan.close()
