"""GPU tests of workspaces that have no room for the leaves' boxes: every step of
every unit is tested, sixteen rounds of steps to an item of work, against the
oracle and against the layout with boxes."""
import numpy as np
import pytest

import oracle
from paper_2005_06773_amd import scenegen as sg
from tests import parity
from tests.test_gpu_box_margins import bytes_without_boxes

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


def _scene(seed, horizon, overlap, outlines):
    rng = np.random.default_rng(seed)
    sides = [(4, 9), (8, 8), (1, 5), (3, 3), (5, 13)]
    objs = [sg.draw_vehicle(rng, 12.0, 0.0, 8.0, *g) for g in sides[:3]]
    objs += [(sg.draw_vehicle if overlap == sg.OVERLAP_PIP else sg.draw_pedestrian)(rng, 12.0, 0.0, 2.0, *g) for g in sides[3:]]
    if outlines:
        objs[0].outline = sg.car_outline(4.4, 1.8)                  # eight corners
        objs[1].outline = sg.random_convex_outline(rng, 4)
        objs[2].outline = sg.random_convex_outline(rng, 7)
    return sg.Scene(objs, horizon, 4.0 / max(horizon, 20), overlap=overlap)


# horizons around a window's 64 and two windows' 128 steps, and odd ones, whose
# units run one to eight steps side by side (1 to 64 rounds)
@pytest.mark.parametrize("overlap,outlines", [(sg.OVERLAP_EXACT, False), (sg.OVERLAP_EXACT, True),
                                              (sg.OVERLAP_PIP, False), (sg.OVERLAP_PIP, True)])
@pytest.mark.parametrize("horizon", [1, 3, 31, 64, 65, 127, 129, 301])
def test_every_step_tested(mhc, ctx, horizon, overlap, outlines):
    s = _scene(horizon, horizon, overlap, outlines)
    cs = mhc.CScene(s)
    c = mhc.mhc_create(0, bytes_without_boxes(mhc, ctx, cs))
    try:
        for v in range(mhc.MHC_N_VARIANTS):
            mhc.mhc_set_variant(c, v)
            got = mhc.mhc_evaluate(c, cs)
            if v == 0:
                parity.check(s, got, oracle.evaluate(s, threads=8), f"H {horizon} overlap {overlap} outlines {outlines}")
            parity.same_results(mhc.mhc_evaluate(ctx, cs), got, f"H {horizon} variant {v}")
    finally:
        mhc.mhc_destroy(c)
