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


def _sharp(angle_deg, reach):
    """A triangle with one corner of angle_deg, `reach` ahead of the tracked
    position, the sharpest that is accepted at 45 degrees."""
    half = math.radians(angle_deg) / 2.0
    h = 1.5 * reach * math.tan(half)
    return np.array([[reach, 0.0], [-0.5 * reach, h], [-0.5 * reach, -h]])


def _corners(o):
    if o.kind != sg.VEHICLE:
        return None
    v = o.outline
    if v is None:
        l, w = o.length / 2.0, o.width / 2.0
        v = np.array([[l, -w], [l, w], [-l, w], [-l, -w]])
    return v


def _half_extent(o, axis):
    """Half of what the object's box covers along an axis (its shape's bounds
    about the tracked position, turned by its heading)."""
    if o.kind != sg.VEHICLE:
        return o.radius
    v = np.abs(_corners(o)).max(axis=0)
    c, s = abs(math.cos(o.heading)), abs(math.sin(o.heading))
    return v[0] * c + v[1] * s if axis == 0 else v[0] * s + v[1] * c


def _near_touch_scene(seed, shift, overlap, sharp):
    """An EGO at (shift, shift) from the scene's origin and shapes all around
    it whose boxes stop 0 to 3 thresholds of the margin away from its box,
    corner towards corner where they have sharp ones."""
    rng = np.random.default_rng(seed)
    ego = _still(sg.VEHICLE, 0.0, 0.0, float(rng.uniform(-math.pi, math.pi)), 1.0, n=2)
    if sharp:
        ego.outline = _sharp(45.5, 2.0)
    objs = [ego]
    margin = 2.0 ** -16 * max(abs(shift), 4.0)
    for k in range(36):
        d = float(rng.choice([0.0, math.pi / 2, math.pi, -math.pi / 2]))     # where it lies
        kind = sg.VEHICLE if overlap == sg.OVERLAP_PIP or k % 3 else sg.PEDESTRIAN
        face = d + math.pi + (float(rng.normal(0.0, 0.02)) if k % 2 else float(rng.uniform(-math.pi, math.pi)))
        o = _still(kind, 0.0, 0.0, face, 0.4 + 0.1 * (k % 5), n=1 + k % 9)
        if kind == sg.VEHICLE and sharp and k % 4:
            o.outline = _sharp(45.2 + k % 3 * 20, 1.0 + 0.5 * (k % 4))
        axis = 0 if abs(math.cos(d)) > 0.5 else 1
        dist = _half_extent(ego, axis) + _half_extent(o, axis) + float(rng.uniform(-0.2, 3.0)) * margin
        side = float(rng.normal(0.0, 0.3))
        o.x = math.cos(d) * dist if axis == 0 else side
        o.y = math.sin(d) * dist if axis == 1 else side
        objs.append(o)
    ego.heading = 0.0 if seed % 2 and sharp else ego.heading
    if shift:
        objs.append(_still(sg.VEHICLE, -2.0 * shift, -2.0 * shift, 0.0, 1.0, n=1))   # puts the origin in between
    return sg.Scene(objs, 2, 0.1, pairs=sg.PAIRS_EGO, overlap=overlap)


@pytest.mark.parametrize("overlap", [sg.OVERLAP_EXACT, sg.OVERLAP_PIP])
@pytest.mark.parametrize("sharp", [False, True])
@pytest.mark.parametrize("shift", [0.0, 3.0e4, 1.0e9])
def test_turned_shapes_at_the_margin(mhc, ctx, shift, sharp, overlap):
    """Turned rectangles, circles and outlines whose sharpest corners are just
    above 45 degrees, in both overlap modes, where the margin decides; far out
    it is wider than the shapes, and their poses are as coarse as the margin."""
    hits = 0
    for seed in range(8):
        s = _near_touch_scene(seed, shift, overlap, sharp)
        got = same_as_testing_every_step(mhc, ctx, s, f"seed {seed} shift {shift} sharp {sharp} overlap {overlap}")
        hits += int((got["first_hit"] >= 0).sum())
    print(f"{hits} colliding pairs", flush=True)
