"""GPU tests of the margin by which two groups' boxes have to lie apart before
the collision kernel leaves a step untested. Every scene is compared with the
same kernel in a workspace that has no room for boxes, which tests every step:
what the boxes decide has to be what the FP32 tests decide."""
import math

import numpy as np
import pytest

from paper_2005_06773_amd import scenegen as sg
from tests import parity

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


def bytes_without_boxes(mhc, ctx, cs):
    """The least workspace the asynchronous call takes, from its refusal of one
    byte: the layout without boxes, to which any boxes would add."""
    import torch
    _, res = mhc.device_result(cs)
    with pytest.raises(mhc.MhcError) as ei:
        mhc.mhc_evaluate_async(ctx, cs, torch.empty(256, dtype=torch.uint8, device="cuda")[:1], res)
    need = int(str(ei.value).split("need ")[1].split()[0])
    boxes = sum((cs.H * ((t + 7) // 8) * 16 + 255) // 256 * 256 for t in cs.T)
    assert boxes > 0 and need + boxes == mhc.mhc_query_sizes(cs)["device_bytes"]
    return need


def same_as_testing_every_step(mhc, ctx, scene, what):
    cs = mhc.CScene(scene)
    c = mhc.mhc_create(0, bytes_without_boxes(mhc, ctx, cs))
    try:
        every = mhc.mhc_evaluate(c, cs)
    finally:
        mhc.mhc_destroy(c)
    parity.same_results(mhc.mhc_evaluate(ctx, cs), every, what)
    return every


def _still(kind, x, y, heading, size, n=3):
    """An object that stays where it is (n trajectories)."""
    veh = kind == sg.VEHICLE
    return sg.SceneObject(kind, x, y, heading, 0.0, 2.0 * size if veh else 0.0, size if veh else 0.0,
                          0.0 if veh else size, np.zeros(n), np.zeros(1), None)


@pytest.mark.parametrize("scale,outline", [(1.0, False), (1e-12, True), (1e-17, False), (1e-20, True), (1e-23, False),
                                           (1e-23, True), (1e-25, False), (1e-25, True), (1e-41, False)])
def test_scenes_so_small_that_squares_underflow(mhc, ctx, scale, outline):
    """Shapes `scale` apart and a fifth of that in size, at the origin: below
    about 1e-22 m the squared distances of the circle tests are 0 in FP32, and
    the tests find overlaps that the boxes must not take away."""
    s = sg.Scene([_still(sg.VEHICLE, 0.0, 0.0, 0.3, 0.2 * scale),
                  _still(sg.VEHICLE, scale, 0.2 * scale, 1.1, 0.2 * scale),
                  _still(sg.PEDESTRIAN, -scale, 0.1 * scale, 0.0, 0.2 * scale),
                  _still(sg.PEDESTRIAN, 0.0, scale, 0.0, 0.2 * scale, n=9)], 3, 0.1)
    if outline:
        s.objects[1].outline = np.array([[math.cos(a), math.sin(a)] for a in np.arange(6) * math.pi / 3]) * 0.2 * scale
    same_as_testing_every_step(mhc, ctx, s, f"scale {scale} outline {outline}")
