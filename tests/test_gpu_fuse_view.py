"""Depth fusion tests each block of the map once, whatever the map's size:
every block is updated on both sides of the launch's sizes (a block, a lane
or a whole workgroup more), f and w as in the oracle, and a frame into a large
map costs little more than into a small one."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import K4, dn, host, intr, to_dev

pytestmark = pytest.mark.gpu


def _view_keys(n):
    """n block keys of 0.8 m, nearest first, in front of the first camera of the small scene."""
    g = np.stack(np.meshgrid(np.arange(-16, 16), np.arange(-8, 8), np.arange(0, 24), indexing="ij"), -1).reshape(-1, 3)
    return g[np.argsort((g ** 2).sum(1), kind="stable")][:n].astype(np.int32)


@pytest.mark.parametrize("nb", [1, 7, 8, 9, 257, 2047, 2048, 2049, 4100, 9000])
def test_every_block_in_view_is_updated(nb):
    D = dn()
    fr = scenes.frames_c1(0, n_frames=2)
    cam = fr.camera
    ov = oracle.OracleVolume(0.1, 0.3, 20.0, nb, 14, 256)
    gv = D.Volume(0.1, 0.3, 20.0, nb, 14, 256, max_points=cam.width * cam.height, max_candidates=1 << 16)
    keys = _view_keys(nb)
    assert ov.insert(keys) == gv.insert_blocks(to_dev(keys)) == nb
    for d, T in zip(fr.depths, fr.poses):
        ov.fuse(d, K4(cam), T)
        gv.fuse_depth(to_dev(d), intr(D, cam), T)
    np.testing.assert_array_equal(host(gv.extract(D.DN_X_W)), ov.w)
    assert np.abs(host(gv.extract(D.DN_X_F)) - ov.f).max() <= 1e-6
    assert (ov.w > 0).any()


def test_a_frame_into_a_large_map():
    """More than 256 blocks for each workgroup of the usual grid: the blocks
    in view get what a small map of them gets, the others nothing; and out of
    view, a block costs the frame less than 60 ps (18 when each is tested
    once, 130 with 16 tests each)."""
    import torch
    D = dn()
    fr = scenes.frames_c1(0, n_frames=1)
    cam = fr.camera
    K, d, T = intr(D, cam), to_dev(fr.depths[0]), fr.poses[0]
    near, n_far = _view_keys(3000), 530000
    k = np.arange(n_far)
    far = np.stack([k % 97, 400 + k // (97 * 97), k // 97 % 97], 1).astype(np.int32)
    keys = np.concatenate([far[:200000], near, far[200000:]])
    vols, ms = [], []
    for c in (near, keys):
        gv = D.Volume(0.1, 0.3, 20.0, len(c), 21, 4096, max_points=cam.width * cam.height, max_candidates=len(c),
                      state16=False)
        assert gv.insert_blocks(to_dev(c), keep_order=True) == len(c)
        gv.fuse_depth(d, K, T)
        vols.append([gv.extract(x) for x in (D.DN_X_F, D.DN_X_W)])
        away = T.copy()
        away[1, 3] -= 5000.0
        best = np.inf
        for _ in range(8):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(50):
                gv.fuse_depth(d, K, away)
            e[1].record()
            torch.cuda.synchronize()
            best = min(best, e[0].elapsed_time(e[1]) / 50)
        ms.append(best)
        assert not torch.equal(vols[-1][1], torch.zeros_like(vols[-1][1]))
        gv.close()
    for small, large in zip(*vols):
        assert torch.equal(small, large[200000:203000])
        assert not large[:200000].any() and not large[203000:].any()
    print(f"a frame out of view: {len(near)} blocks {1e3 * ms[0]:.2f} us, {len(keys)} blocks {1e3 * ms[1]:.2f} us")
    assert (ms[1] - ms[0]) * 1e9 / n_far < 60.0
