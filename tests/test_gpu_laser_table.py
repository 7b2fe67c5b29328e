"""Laser fusion through the table of the blocks that a workgroup met, which
serves maps of 4097 to 16384 blocks and rays that reach beyond 500 blocks:
weights exact and f within 1e-5 of the oracle, with entries that replace each
other, blocks that are not allocated, and blocks past the table's range."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import dn, host, to_dev

pytestmark = pytest.mark.gpu


def _pair(s, mu, far, cap, n, **kw):
    D = dn()
    ov = oracle.OracleVolume(s, mu, far, cap, 16, 512)
    gv = D.Volume(s, mu, far, cap, 16, 512, max_points=n, state16=False,
                  max_observations=kw.pop("max_observations", D.laser_observations_bound(n, s, mu, far)), **kw)
    return D, ov, gv


def _scan(D, ov, gv, pts, T):
    assert ov.alloc_laser(pts, T) == gv.alloc_laser(to_dev(pts), T)
    ov.fuse_laser(pts, T)
    gv.fuse_laser(to_dev(pts), T)
    assert gv.num_blocks == ov.nb
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_W)), ov.w)
    assert np.abs(host(gv.extract(D.DN_X_F)) - ov.f).max() <= 1e-5


# blocks before the scans: the smallest and largest maps of the table (the
# scans add about 500), with a box of blocks around the sensor that most rays
# run through
@pytest.mark.parametrize("before", [4097, 5000, 12000, 15500])
@pytest.mark.parametrize("returns", [1, 257, 4097])
def test_maps_past_the_whole_table(before, returns):
    D, ov, gv = _pair(0.1, 0.3, 20.0, 1 << 14, 1 << 13)
    k = np.arange(before)
    keys = np.stack([k % 32 - 16, (k // 32) % 16 - 8, k // 512 - 8], 1).astype(np.int32)
    assert ov.insert(keys) == gv.insert_blocks(to_dev(keys)) == before
    for j in range(2):
        T = scenes.pose_yaw(0.1 * j, 0.05 + 0.3 * j, -0.1, 0.7 * j)
        pts = scenes.laser_scan(scenes.scene_c1(), T, j, n_rings=16, n_azimuth=257)
        if returns < 4097:
            pts = pts[np.isfinite(pts[:, 0])]
        _scan(D, ov, gv, pts[np.linspace(0, len(pts) - 1, returns).astype(int)], T)
    assert 4096 < gv.num_blocks <= 16384 and (ov.w > 0).sum() > 100


def test_returns_past_the_range_of_the_table():
    """8 cm blocks and returns up to 48 m: 600 blocks from the sensor, on
    both sides of the table's 512, along the axes and between them."""
    n = 64
    D, ov, gv = _pair(0.01, 0.03, 50.0, 1 << 12, n)
    rng = np.random.default_rng(4)
    d = np.concatenate([np.eye(3), -np.eye(3), rng.normal(size=(n - 6, 3))])
    d /= np.linalg.norm(d, axis=1)[:, None]
    pts = (d * np.linspace(36.0, 48.0, n)[:, None]).astype(np.float32)
    _scan(D, ov, gv, pts, scenes.pose_yaw(0.1, 0.3, -0.1, 0.7))
    assert np.abs(ov.coords).max() > 530 and (ov.w > 0).sum() > 64
