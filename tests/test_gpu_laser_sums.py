"""The sums of a laser scan keep the digits of float64, whatever the number of
returns they are sized for: many returns of one voxel whose distances to the
surface nearly cancel or are tiny, against exact rational sums."""
from fractions import Fraction

import numpy as np
import pytest

from gpu_common import dn, host, to_dev

pytestmark = pytest.mark.gpu

S, MU, FAR = 0.125, 0.375, 20.0       # (binary fractions: the geometry below is exact)


def _eta(z):
    """eta / mu of a return at depth z along +z for the voxels of its column, float64 as the walk evaluates it."""
    z = np.asarray(z, np.float32).astype(np.float64)
    k = np.arange(0, 200)
    eta = z[:, None] - (k + 0.5) * S
    ok = (eta >= -MU) & (k * S <= z[:, None] + MU)
    return ok, np.minimum(1.0, eta / MU)


@pytest.mark.parametrize("padding", [0, 1 << 16, 1 << 20])
@pytest.mark.parametrize("case", ["tiny", "cancelling", "many", "end of the band"])
def test_sums_keep_the_digits_of_float64(case, padding):
    D = dn()
    centre, up = 10.5 * S, 2.0 ** -23         # up: one step of float32 there
    z = {"tiny": [centre + up], "cancelling": [centre + 3 * up, centre - 2 * up, centre - up, centre + up],
         "many": centre + up * (np.arange(4001) % 7 - 3),
         "end of the band": np.full(130, centre)}[case]        # psi = -1 exactly in voxel 13, in whole waves
    z = np.asarray(z, np.float32)
    # padding: more returns (not valid ones) of the same scan
    pts = np.full((len(z) + padding, 3), np.nan, np.float32)
    at = np.arange(len(z)) * (len(pts) // len(z))
    pts[at] = 0
    pts[at, 2] = z
    T = np.eye(4)
    T[:3, 3] = (0.5 * S, 0.5 * S, 0.0)
    gv = D.Volume(S, MU, FAR, 64, 8, 64, max_points=len(pts), max_candidates=max(1 << 16, 8 * len(z)),
                  max_observations=1 << 21, state16=False)
    gv.alloc_laser(to_dev(pts), T)
    gv.insert_blocks(to_dev(np.array([[0, 0, 0], [0, 0, 1], [0, 0, 2]], np.int32)))
    gv.fuse_laser(to_dev(pts), T)
    coords, f, w = (host(gv.extract(k)) for k in (D.DN_X_COORDS, D.DN_X_F, D.DN_X_W))
    ok, psi = _eta(z)
    checked = 0
    for b, c in enumerate(coords):
        if c[0] or c[1]:
            continue
        for v in range(8):
            k = 8 * c[2] + v
            n = int(ok[:, k].sum())
            assert w[b, 64 * v] == n
            if n == 0:
                continue
            total = sum((Fraction(float(x)) for x in psi[ok[:, k], k]), Fraction(0))
            want = float(total / n)
            # float64 sums of n terms, and the rounding to float32
            tol = abs(want) * 2.0 ** -24 * 1.001 + float(np.abs(psi[ok[:, k], k]).sum()) * 2.0 ** -53
            assert abs(float(f[b, 64 * v]) - want) <= tol, (k, f[b, 64 * v], want)
            checked += 1
    assert checked >= 12
