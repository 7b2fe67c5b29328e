"""Every form of the fused iteration (8, 4, 2 or 1 waves per block, in pool
or Morton order) computes each voxel with the same operations: what the
tuner picks equals the explicit 512- and 256-thread kernels bit for bit, in
FP32 and 16-bit state, on sparse block sets (unallocated and unobserved
neighbours on every side), and the FP32 result agrees with the two-pass
kernels, which use the compiler's own square root and division."""
import numpy as np
import pytest

import scenes
from gpu_common import LAM, dn, host, state_of, to_dev

pytestmark = pytest.mark.gpu


def _volume(D, nb, extent):
    coords, f, w = scenes.random_block_field(nb, 5, extent=extent, omega_frac=0.7)
    gv = D.Volume(0.1, 0.3, 10.0, nb, 14, 256, max_points=0, max_candidates=max(nb, 64))
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    gv.load_fused(to_dev(f.astype(np.float32)), to_dev(w.astype(np.float32)))
    return gv


@pytest.mark.parametrize("nb,extent", [(1, 1), (2, 2), (65, 5), (513, 9), (6000, 20)])
@pytest.mark.parametrize("storage", ["DN_F32", "DN_F16", "DN_BF16"])
@pytest.mark.parametrize("data", ["DN_DATA_L2", "DN_DATA_L1"])
def test_every_form_gives_the_same_bits(nb, extent, storage, data):
    D = dn()
    gv = _volume(D, nb, extent)
    got = []
    for kernel in (D.DN_K_AUTO, D.DN_K_AUTO, D.DN_K_FUSED, D.DN_K_FUSED256):
        st = gv.regularize(D.reg_params(LAM, iters=23, kernel=kernel, storage=getattr(D, storage), refine_every=7,
                                        data_term=getattr(D, data)))
        got.append(state_of(D, gv))
        print(f"{storage} {nb} blocks: asked {kernel}, ran {st.kernel_used} layout {st.layout_used}")
    for other in got[1:]:
        for a, b in zip(got[0], other):
            np.testing.assert_array_equal(a, b)
    if storage == "DN_F32":
        gv.regularize(D.reg_params(LAM, iters=23, kernel=D.DN_K_TWOPASS, data_term=getattr(D, data)))
        for a, b in zip(got[0], state_of(D, gv)):
            assert np.abs(a - b).max() <= 1e-5


def test_huge_weights_and_duals_take_the_general_division():
    """Weights up to 1e38 (the quotient's denominator beyond 2^96) and a
    given dual state far outside the unit ball: the same values as the
    two-pass kernels, finite where theirs are."""
    D = dn()
    gv = _volume(D, 9, 3)
    w = host(gv.extract(D.DN_X_W))
    f = host(gv.extract(D.DN_X_F))
    w[:, ::3] *= np.float32(1e37)
    gv.load_fused(to_dev(f), to_dev(w))
    p0 = np.random.default_rng(0).normal(size=(3, 9, 512)).astype(np.float32) * np.float32(1e15)
    out = []
    for kernel in (D.DN_K_FUSED, D.DN_K_TWOPASS):
        try:
            gv.regularize(D.reg_params(LAM, iters=3, kernel=kernel, init=D.DN_INIT_GIVEN), to_dev(f), to_dev(p0))
        except D.DenserError as e:
            assert e.code == D.DN_E_NUMERIC
        out.append(state_of(D, gv))
    for a, b in zip(*out):
        assert np.array_equal(np.isfinite(a), np.isfinite(b))
        ok = np.isfinite(a)
        np.testing.assert_allclose(a[ok], b[ok], rtol=1e-5, atol=1e-5)
