"""The serving scheduler's admission, on the CPU: a frame is taken wherever its
workspace without the leaves' boxes fits with room for its vehicles' poses once
more, and what is reserved for it covers the workspace it then gets."""
import numpy as np
import pytest

from paper_2005_06773_amd import scenegen as sg


@pytest.fixture(scope="module")
def mhc():
    from paper_2005_06773_amd import mhc as m
    return m


def _objects(n_veh, n_ped, side, seed=3):
    rng = np.random.default_rng(seed)
    objs = [sg.draw_vehicle(rng, 30.0, 0.0, 15.0, side, side) for _ in range(n_veh)]
    return objs + [sg.draw_pedestrian(rng, 30.0, 0.0, 2.0, side, side) for _ in range(n_ped)]


# the bytes of a slot that admission leaves out
RESERVE = (1 << 18) + 256


def _least_slot(mhc, scene):
    """The least budget of a one-slot server that takes the frame (first hits
    asked for), less what admission leaves out of a slot."""
    start = 2 * RESERVE + 256        # a server takes a larger budget only
    lo, hi = start, 1 << 34
    while hi - lo > 256:
        mid = (lo + hi) // 2 // 256 * 256
        srv = mhc.Server(None, executor=(lambda *a: 0, lambda *a: 1), inflight=1, budget=mid)
        try:
            srv.submit(0, scene, first_hit=True)
            hi = mid
        except mhc.MhcError as e:
            assert e.status == mhc.MHC_E_NOMEM
            lo = mid
        finally:
            srv.stop()
    assert lo > start
    return hi - RESERVE


# objects of one trajectory, whose boxes take as much as a vehicle's poses and
# twice a pedestrian's; a street with and without a crowd; outlines; risk over time
@pytest.mark.parametrize("n_veh,n_ped,side,horizon,option", [
    (1, 7, 1, 30000, ""), (1, 1, 1, 32000, ""), (0, 9, 1, 20000, ""), (1, 30, 15, 100, "ego"), (6, 5, 15, 30, ""),
    (2, 14, 3, 2000, ""), (6, 5, 12, 40, "outlines"), (3, 3, 9, 60, "timeline")])
def test_boxes_take_no_more_than_vehicles_poses(mhc, n_veh, n_ped, side, horizon, option):
    s = sg.Scene(_objects(n_veh, n_ped, side), horizon, 0.01, pairs=sg.PAIRS_EGO if option == "ego" else sg.PAIRS_ALL)
    if option == "outlines":
        for o in s.objects[:n_veh]:
            o.outline = sg.car_outline(o.length, o.width)
    s.timeline = int(option == "timeline")
    cs = mhc.CScene(s)
    boxes = sum((cs.H * ((t + 7) // 8) * 16 + 255) // 256 * 256 for t in cs.T)
    least = mhc.mhc_query_sizes(cs)["device_bytes"] - boxes       # the workspace without boxes
    got = _least_slot(mhc, s)
    assert got >= least, (got, least)
    # the bound's slack: 16 tables of alignment, trajectory kernel rows and polygons it may not need
    rows = sum((t + 7) // 8 + 1 for t in cs.T) * 8
    poses = sum((cs.H * t * 16 + 255) // 256 * 256 for t in cs.T[:n_veh])
    assert got <= least + (boxes if boxes <= poses else 0) + 36 * 256 + rows + len(cs.T) * 512, (got, least, boxes, poses)
