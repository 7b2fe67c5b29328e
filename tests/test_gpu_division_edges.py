"""The fused iteration's short square root and division give the bits of the
two-pass kernels, which use the compiler's general ones, at the ends of the
exponent range too: subnormal and tiny fields and duals, numerators around the
line between the short and the general path, large weights, infinite values."""
import numpy as np
import pytest

import scenes
from gpu_common import LAM, dn, host, state_of, to_dev

pytestmark = pytest.mark.gpu

NB = 40


def _volume(D):
    coords, f, w = scenes.random_block_field(NB, 5, extent=4, omega_frac=0.7)
    gv = D.Volume(0.1, 0.3, 10.0, NB, 10, 256, max_points=0, max_candidates=64)
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    return gv, np.asarray(w, np.float32).reshape(NB, 512)


def _spread(rng, shape, lo, hi):
    """Both signs, magnitudes spread over [2^lo, 2^hi], some zeros of both signs."""
    x = np.ldexp(1.0 + rng.random(shape), rng.integers(lo, hi, shape)) * rng.choice([-1.0, 1.0], shape)
    return np.where(rng.random(shape) < 0.1, np.copysign(0.0, x), x).astype(np.float32)


def _both(D, gv, f, w, u0, p0, iters):
    gv.load_fused(to_dev(f), to_dev(w))
    out = []
    for kernel in (D.DN_K_TWOPASS, D.DN_K_FUSED, D.DN_K_FUSED256):
        try:
            gv.regularize(D.reg_params(LAM, iters=iters, kernel=kernel, init=D.DN_INIT_GIVEN), to_dev(u0), to_dev(p0))
        except D.DenserError as e:
            assert e.code == D.DN_E_NUMERIC
        out.append([x.astype(np.float32) for x in state_of(D, gv)])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            np.testing.assert_array_equal(a, b)
    return out[0]


@pytest.mark.parametrize("lo,hi", [(-149, -120), (-127, -90), (-104, -96), (-104, 1)])
@pytest.mark.parametrize("weights", [1.0, 2.0 ** 20, 2.0 ** 27, 2.0 ** 60])
def test_tiny_fields(lo, hi, weights):
    """(weights: denominators on both sides of 2^24)"""
    D = dn()
    gv, w = _volume(D)
    rng = np.random.default_rng(-lo)
    f, u0 = (_spread(rng, (NB, 512), lo, hi) for _ in range(2))
    u, _, _ = _both(D, gv, f, w * np.float32(weights), u0, np.zeros((3, NB, 512), np.float32), 3)
    assert np.isfinite(u).all() and (u != u0).any()


@pytest.mark.parametrize("scale", [0, 23, 24, 47, 50])
def test_duals_with_tiny_components(scale):
    """One component of magnitude 2^scale to 2^(scale + 1), the others tiny."""
    D = dn()
    gv, w = _volume(D)
    rng = np.random.default_rng(scale)
    p0 = _spread(rng, (3, NB, 512), -149, -60)
    big = np.ldexp(1.0 + rng.random((NB, 512)), scale).astype(np.float32)
    np.put_along_axis(p0, rng.integers(0, 3, (1, NB, 512)), big[None], 0)
    zero = np.zeros((NB, 512), np.float32)
    _, _, p = _both(D, gv, zero, w, zero, p0, 1)
    assert (np.abs(p).max(0) == 1.0).mean() > 0.5 and ((p != 0) & (np.abs(p) < 2.0 ** -80)).any()


def test_infinite_values_stay_infinite():
    D = dn()
    gv, w = _volume(D)
    rng = np.random.default_rng(7)
    f = _spread(rng, (NB, 512), -4, 1)
    f[:, 3::97] = np.inf
    f[:, 5::89] = -np.inf
    f[:, 7::83] = np.float32(3e38)
    u, _, _ = _both(D, gv, f, w, np.zeros_like(f), np.zeros((3, NB, 512), np.float32), 1)
    seen = (w > 0) & np.isinf(f)
    assert seen.any() and (u[seen] == f[seen]).all()
