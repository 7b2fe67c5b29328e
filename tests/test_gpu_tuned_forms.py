"""Every form of the iteration that the tuner can pick (8, 4, 2 and 1 waves per
block, in Morton and in pool order) gives the bits of the explicit 8-wave
kernel, off the observed voxels too: in FP32 and 16-bit state, on small maps
and on ones beyond the caches, where lines without an observed voxel rest, from
zero, kept and given states.  The tuner's memory is set to each form in turn."""
import ctypes

import numpy as np
import pytest

import scenes
from gpu_common import LAM, dn, state_of, to_dev

pytestmark = pytest.mark.gpu

FORMS = [(kernel, layout) for kernel in (2, 3, 4, 5) for layout in (0, 1)]


def _choose(D, gv, storage, kernel, layout):
    fn = D.lib()["_ZN2dn15remember_choiceEPK9dn_volumeiii"]
    fn.argtypes, fn.restype = [ctypes.c_void_p] + 3 * [ctypes.c_int], None
    fn(gv.handle, storage, kernel, layout)


def _volume(D, nb, extent):
    coords, f, w = scenes.random_block_field(nb, 5, extent=extent, omega_frac=0.7)
    w = np.asarray(w, np.float32).reshape(nb, 512).copy()
    rng = np.random.default_rng(nb)
    w[rng.random(nb) < 0.2] = 0
    w.reshape(-1, 32)[rng.random(nb * 16) < 0.3] = 0
    gv = D.Volume(0.1, 0.3, 10.0, nb, 16, 256, max_points=0, max_candidates=max(nb, 64))
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    gv.load_fused(to_dev(np.asarray(f, np.float32).reshape(nb, 512)), to_dev(w))
    return gv, to_dev(np.asarray(f, np.float32).reshape(nb, 512)), w


def _solves(D, gv, storage, kernel, data, f, p0, form=None):
    """The states after a solve from zero, a kept one and a given one, and what ran."""
    out, ran = [], []
    for init, iters, given in ((D.DN_INIT_ZERO, 9, ()), (D.DN_INIT_KEEP, 4, ()), (D.DN_INIT_GIVEN, 6, (f, p0))):
        if form:
            _choose(D, gv, storage, *form)
        st = gv.regularize(D.reg_params(LAM, iters=iters, kernel=kernel, storage=storage, refine_every=4, init=init,
                                        data_term=data), *given)
        out.append(state_of(D, gv))
        ran.append((st.kernel_used, st.layout_used))
    return out, ran


SMALL = [(s, nb, extent) for s in ("DN_F32", "DN_F16", "DN_BF16") for nb, extent in ((1, 1), (65, 5), (513, 9))]


@pytest.mark.parametrize("storage,nb,extent", SMALL + [("DN_F32", 13001, 26), ("DN_BF16", 21001, 31)])
def test_every_form_the_tuner_can_pick(storage, nb, extent):
    D = dn()
    gv, f, w = _volume(D, nb, extent)
    p0 = np.random.default_rng(3).normal(size=(3, nb, 512)).astype(np.float32)
    p0[:, w == 0] = 0
    p0, storage = to_dev(p0), getattr(D, storage)
    try:
        for data in (D.DN_DATA_L2, D.DN_DATA_L1):
            want, _ = _solves(D, gv, storage, D.DN_K_FUSED, data, f, p0)
            for form in FORMS:
                got, ran = _solves(D, gv, storage, D.DN_K_AUTO, data, f, p0, form)
                assert ran == [form] * 3
                for a, b in zip(want, got):
                    for x, y in zip(a, b):
                        np.testing.assert_array_equal(x, y)
    finally:
        _choose(D, gv, storage, D.DN_K_FUSED256, 0)
        gv.close()
