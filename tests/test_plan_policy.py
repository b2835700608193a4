"""The collision plans that the wave counts of a whole GPU lead to, walked on the
host: every trajectory pair in one item of one unit."""
import numpy as np
import pytest

from paper_2005_06773_amd import scenegen as sg

# resident waves of the collision kernel on 256 CUs: rectangles and circles,
# and outlines; and 4/5 of them, which a large server tick plans for
WAVES = {False: (6144, 4912), True: (4096, 3272)}


@pytest.fixture(scope="module")
def mhc():
    from paper_2005_06773_amd import mhc as m
    return m


def _objects(n, side, outlines):
    rng = np.random.default_rng(n * 100 + side)
    objs = [sg.draw_vehicle(rng, 30.0, 0.0, 20.0, side, side) for _ in range(n)]
    if outlines:
        for o in objs:
            o.outline = sg.car_outline(o.length, o.width)
    return sg.Scene(objs, 30, 0.1)


# around one block a wave with sides of 8 and of 16, and half of one with 32
@pytest.mark.parametrize("outlines", [False, True])
@pytest.mark.parametrize("n,side", [(2, 5), (3, 13), (6, 13), (9, 11), (12, 9), (16, 7), (20, 7), (20, 11), (11, 15), (24, 20)])
def test_plans_of_a_whole_gpu_cover_every_pair(mhc, n, side, outlines):
    s = _objects(n, side, outlines)
    for waves in WAVES[outlines]:
        for v in range(mhc.MHC_N_VARIANTS):
            st, info = mhc.mhc_plan_check(s, v, waves)
            assert st == mhc.MHC_OK, (waves, v, info)
            # units of one pair of leaves, 8 steps of an item side by side; a
            # unit of outlines' single pairs holds 32 at 2 steps
            assert info["time_split"] == (2 if outlines else 8), (waves, v, info)


@pytest.mark.parametrize("n,side", [(16, 7), (12, 9), (20, 7), (9, 11), (6, 13)])
def test_smallest_blocks_only_while_no_wave_looks_twice(mhc, n, side):
    """Plans of 0.96 to 1.5 blocks of side 8 a wave take one round of looks."""
    st, info = mhc.mhc_plan_check(_objects(n, side, False), 0, 6144)
    assert st == mhc.MHC_OK and info["contiguous"] == 0, info


@pytest.mark.parametrize("n,side,outlines,workgroups", [(6, 5, False, 240), (6, 5, True, 240), (12, 9, False, 384),
                                                        (8, 7, True, 512), (2, 1, True, 1), (2, 1, False, 1)])
def test_few_strips_go_to_many_workgroups(mhc, n, side, outlines, workgroups):
    """One strip a workgroup while there are no more than half of those that
    the GPU holds, for outlines all of them."""
    st, info = mhc.mhc_plan_check(_objects(n, side, outlines), 0, WAVES[outlines][0])
    assert st == mhc.MHC_OK and info["n_waves"] == workgroups * 8, info
