"""Allocation and laser fusion over the sizes where the library changes its
path: frames with few and with many new blocks, into empty, small, larger
and very large maps, through explicit insertions in between, near the end of
the hash table's tail, and scans into maps on both sides of the accumulator
limit.  Block keys, pool order, hash slots and the neighbour table are bit-
exact against the oracle, weights exact, f within 1e-5."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import K4, dn, host, intr, to_dev

pytestmark = pytest.mark.gpu


def _check(D, ov, gv):
    assert gv.num_blocks == ov.nb
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_COORDS)), ov.coords)
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_HASH)), ov.slots)
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_NBR)), ov.nbr)


def _grid(n, origin):
    """n block keys in a box far from the scene."""
    e = int(np.ceil(n ** (1 / 3)))
    k = np.arange(n)
    return (np.stack([k % e, (k // e) % e, k // (e * e)], 1) + np.asarray(origin)).astype(np.int32)


# (voxel size, blocks in the map beforehand): few new blocks a frame into maps whose merge stays in LDS / goes
# through memory / takes the general insertion; more than 4096 new blocks in the first frame
@pytest.mark.parametrize("voxel,before", [(0.1, 0), (0.1, 3000), (0.1, 9000), (0.1, 66000), (0.02, 0), (0.02, 500)])
def test_frames_into_maps_of_every_size(voxel, before):
    D = dn()
    fr = scenes.frames_c1(0, n_frames=3)
    cam = fr.camera
    cap = 1 << 17
    ov = oracle.OracleVolume(voxel, 3 * voxel, fr.max_depth, cap, 18, 512)
    gv = D.Volume(voxel, 3 * voxel, fr.max_depth, cap, 18, 512, max_points=cam.width * cam.height,
                  max_candidates=1 << 20, state16=False)
    K = intr(D, cam)
    if before:
        keys = _grid(before, (-40, -300, -40))
        assert ov.insert(keys) == gv.insert_blocks(to_dev(keys))
    for k, (d, T) in enumerate(zip(fr.depths, fr.poses)):
        n_o = ov.alloc(d, K4(cam), T)
        assert n_o == gv.alloc_blocks(to_dev(d), K, T)
        np.testing.assert_array_equal(host(gv.extract(D.DN_X_CANDIDATES)), ov.last_candidates)
        _check(D, ov, gv)
        print(f"voxel {voxel}, {before} before, frame {k}: {n_o} new")
    # an explicit insertion, then a frame again
    keys = _grid(100, (30, 30, 30))
    assert ov.insert(keys) == gv.insert_blocks(to_dev(keys))
    T = scenes.pose_yaw(0.3, 0.5, 0.0, 0.5)
    assert ov.alloc(fr.depths[0], K4(cam), T) == gv.alloc_blocks(to_dev(fr.depths[0]), K, T)
    _check(D, ov, gv)
    gv.clear()
    assert gv.alloc_blocks(to_dev(fr.depths[0]), K, fr.poses[0]) > 0


def test_full_pool_and_full_table_leave_the_map_as_it_was():
    """A frame that does not fit the pool, one whose band cells exceed
    max_candidates and one that overflows the table's short tail are
    refused; the map stays, and a later frame that fits is taken."""
    D = dn()
    fr = scenes.frames_c1(0, n_frames=2)
    cam = fr.camera
    K = intr(D, cam)
    d = to_dev(fr.depths[0])
    empty = to_dev(np.zeros((cam.height, cam.width), np.float32))
    few = np.zeros((cam.height, cam.width), np.float32)
    few[40:50, 150:170] = fr.depths[0][40:50, 150:170]
    for kw in (dict(max_blocks=60, log2=12, tail=256), dict(max_blocks=4096, log2=4, tail=60),
               dict(max_blocks=4096, log2=12, tail=256, max_candidates=2000)):
        kw = dict(kw)
        mc = kw.pop("max_candidates", 1 << 18)
        ov = oracle.OracleVolume(0.1, 0.3, 20.0, kw["max_blocks"], kw["log2"], kw["tail"])
        gv = D.Volume(0.1, 0.3, 20.0, kw["max_blocks"], kw["log2"], kw["tail"], max_points=cam.width * cam.height,
                      max_candidates=mc)
        assert ov.alloc(few, K4(cam), fr.poses[0]) == gv.alloc_blocks(to_dev(few), K, fr.poses[0])
        _check(D, ov, gv)
        for _ in range(2):
            with pytest.raises(D.DenserError) as e:
                gv.alloc_blocks(d, K, fr.poses[0])
            assert e.value.code == D.DN_E_CAPACITY
            _check(D, ov, gv)
        assert gv.alloc_blocks(empty, K, fr.poses[0]) == 0
        few2 = np.roll(few, 40, axis=1)
        assert ov.alloc(few2, K4(cam), fr.poses[0]) == gv.alloc_blocks(to_dev(few2), K, fr.poses[0])
        _check(D, ov, gv)


@pytest.mark.parametrize("before", [0, 16384])
@pytest.mark.parametrize("returns", [1, 63, 4097])
def test_scans_on_both_sides_of_the_accumulator_limit(before, returns):
    D = dn()
    boxes = scenes.scene_c1()
    cap, s, mu = 1 << 15, 0.1, 0.3
    ov = oracle.OracleVolume(s, mu, 20.0, cap, 16, 512)
    gv = D.Volume(s, mu, 20.0, cap, 16, 512, max_points=1 << 13, state16=False,
                  max_observations=D.laser_observations_bound(1 << 13, s, mu, 20.0))
    if before:
        keys = _grid(before, (-40, -300, -40))
        assert ov.insert(keys) == gv.insert_blocks(to_dev(keys))
    for k in range(2):
        T = scenes.pose_yaw(0.1 * k, 0.05 + 0.3 * k, -0.1, 0.7 * k)
        pts = scenes.laser_scan(boxes, T, k, n_rings=16, n_azimuth=257)
        if returns < 4097:
            pts = pts[np.isfinite(pts[:, 0])]
        pts = pts[np.linspace(0, len(pts) - 1, returns).astype(int)]
        assert ov.alloc_laser(pts, T) == gv.alloc_laser(to_dev(pts), T)
        ov.fuse_laser(pts, T)
        gv.fuse_laser(to_dev(pts), T)
        _check(D, ov, gv)
        np.testing.assert_array_equal(host(gv.extract(D.DN_X_W)), ov.w)
        assert np.abs(host(gv.extract(D.DN_X_F)) - ov.f).max() <= 1e-5


def test_a_scan_with_too_many_observations_changes_nothing():
    D = dn()
    T = scenes.pose_yaw(0.1, 0.0, 0.0, 0.0)
    pts = to_dev(scenes.laser_scan(scenes.scene_c1(), T, 1))
    full = D.Volume(0.1, 0.3, 20.0, 4096, 12, 256, max_points=1 << 13, max_observations=1 << 20)
    gv = D.Volume(0.1, 0.3, 20.0, 4096, 12, 256, max_points=1 << 13, max_observations=1000)
    for v in (full, gv):
        v.alloc_laser(pts, T)
    full.fuse_laser(pts, T)
    with pytest.raises(D.DenserError) as e:
        gv.fuse_laser(pts, T)
    assert e.value.code == D.DN_E_CAPACITY
    assert not host(gv.extract(D.DN_X_W)).any() and host(full.extract(D.DN_X_W)).any()


def test_counts_come_back_with_and_without_a_report_buffer():
    """The same counts through the caller's pinned words and through copies;
    ordinary memory is refused."""
    import ctypes
    D = dn()
    fr = scenes.frames_c1(0, n_frames=2)
    cam = fr.camera
    K = intr(D, cam)
    gv = D.Volume(0.1, 0.3, 20.0, 4096, 12, 256, max_points=cam.width * cam.height, **{"max_observations": 1 << 21})
    pts = to_dev(scenes.laser_scan(scenes.scene_c1(), fr.poses[0], 1))
    got = []
    for buffer in (True, False):
        gv.clear()
        if not buffer:
            D.check(D.lib().dn_set_report_buffer(gv.handle, None, 0))
        n = [gv.integrate(to_dev(d), K, T) for d, T in zip(fr.depths, fr.poses)]
        n.append(gv.integrate_laser(pts, fr.poses[0]))
        got.append((n, host(gv.extract(D.DN_X_W)), host(gv.extract(D.DN_X_F))))
    assert got[0][0] == got[1][0]
    for a, b in zip(got[0][1:], got[1][1:]):
        np.testing.assert_array_equal(a, b)
    plain = (ctypes.c_int64 * 8)()
    assert D.lib().dn_set_report_buffer(gv.handle, ctypes.cast(plain, ctypes.c_void_p), 64) == D.DN_E_INVALID
    assert gv.integrate(to_dev(fr.depths[0]), K, fr.poses[0]) == 0
