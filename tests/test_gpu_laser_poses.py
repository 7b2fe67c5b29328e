"""Scans whose pose is not rigid (a scaled, stretched, sheared or mirrored
sensor frame): eta = r - (c - o) . D is evaluated as for any other pose, so
weights are exact and f is within 1e-5 of the oracle."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import dn, host, to_dev

pytestmark = pytest.mark.gpu

FRAMES = {"half": np.eye(3) * 0.5, "near rigid": np.eye(3) * 1.001, "larger": np.eye(3) * 1.7,
          "stretched": np.diag([0.6, 1.0, 1.5]), "mirrored": np.diag([1.0, 1.0, -1.0]),
          "sheared": np.array([[1.0, 0.4, 0.0], [0.0, 1.0, 0.3], [0.2, 0.0, 1.0]])}


def _compare(s, mu, far, pts, T):
    D = dn()
    ov = oracle.OracleVolume(s, mu, far, 1 << 13, 16, 512)
    gv = D.Volume(s, mu, far, 1 << 13, 16, 512, max_points=len(pts), state16=False, max_candidates=1 << 20,
                  max_observations=4 * D.laser_observations_bound(len(pts), s, mu, far))
    # the blocks along the way too, so that free space is observed
    near = np.concatenate([oracle.candidates_laser(pts[::7] * np.float32(a), T, s, mu, far) for a in (0.15, 0.3)])
    assert ov.insert(near) == gv.insert_blocks(to_dev(near))
    for _ in range(2):
        assert ov.alloc_laser(pts, T) == gv.alloc_laser(to_dev(pts), T)
        ov.fuse_laser(pts, T)
        gv.fuse_laser(to_dev(pts), T)
    assert gv.num_blocks == ov.nb <= 4096
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_W)), ov.w)
    assert np.abs(host(gv.extract(D.DN_X_F)) - ov.f).max() <= 1e-5
    return ov


@pytest.mark.parametrize("name", FRAMES)
def test_poses_that_are_not_rigid(name):
    rigid = scenes.pose_yaw(0.1, 0.3, -0.1, 0.7)
    T = rigid.copy()
    T[:3, :3] = rigid[:3, :3] @ FRAMES[name]
    pts = scenes.laser_scan(scenes.scene_c1(), rigid, 2, n_rings=12, n_azimuth=180)
    ov = _compare(0.1, 0.3, 20.0, pts, T)
    assert (ov.w > 0).sum() > 1000


@pytest.mark.parametrize("scale", [0.7, 1.0, 2.2])
def test_rays_that_reach_further_than_their_range(scale):
    """16 cm blocks, ranges up to 313 of them, seen at up to 688."""
    rng = np.random.default_rng(4)
    d = np.concatenate([np.eye(3), -np.eye(3), rng.normal(size=(58, 3))])
    d /= np.linalg.norm(d, axis=1)[:, None]
    T = scenes.pose_yaw(0.1, 0.3, -0.1, 0.7)
    T[:3, :3] *= scale
    ov = _compare(0.02, 0.06, 50.0, (d * np.linspace(20.0, 49.0, 64)[:, None]).astype(np.float32), T)
    assert (ov.w > 0).any()
