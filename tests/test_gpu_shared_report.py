"""Volumes that report to the same page-locked words: a batched solve still
gives each its own energies, as volumes with words of their own get them and
those without any."""
import ctypes

import pytest

import scenes
from gpu_common import LAM, dn, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [0, 8, 64, None])
def test_batched_energies_of_volumes_that_share_a_report_buffer(step):
    """step: bytes from one volume's buffer to the next (None: no buffers)."""
    import torch
    D = dn()
    sizes = (40, 90, 7)
    vols = []
    for k, n in enumerate(sizes):
        coords, f, w = scenes.random_block_field(n, 5 + k, extent=6, omega_frac=0.7)
        gv = D.Volume(0.1, 0.3, 10.0, n, 10, 256, max_points=0, max_candidates=128)
        gv.insert_blocks(to_dev(coords.astype("int32")), keep_order=True)
        gv.load_fused(to_dev(f.astype("float32")), to_dev(w.astype("float32")))
        vols.append(gv)
    prm = D.reg_params(LAM, iters=11, kernel=D.DN_K_FUSED256)
    want = [(s.energy, s.dual) for s in D.regularize_batch(vols, prm)]
    assert len(set(want)) == len(sizes)
    words = torch.empty(512, dtype=torch.uint8, pin_memory=True)
    for k, gv in enumerate(vols):
        at = ctypes.c_void_p(words.data_ptr() + k * step) if step is not None else None
        D.check(D.lib().dn_set_report_buffer(gv.handle, at, 64 if at else 0))
    assert [(s.energy, s.dual) for s in D.regularize_batch(vols, prm)] == want
    for gv in vols:
        gv.close()
