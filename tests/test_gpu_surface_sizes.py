"""Surface points, mesh, area and energies over the sizes where their
reductions and scans change (one workgroup up to 16384 pairs / 32768 blocks,
device-wide beyond), on random fields with every neighbour pattern, against
the oracle on the same float field."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import LAM, dn, host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,extent", [(1, 1), (300, 8), (4097, 20), (16385, 30), (33000, 36)])
def test_surface_mesh_and_energy_of_random_fields(nb, extent):
    D = dn()
    coords, f, w = scenes.random_block_field(nb, 3, extent=extent, omega_frac=0.5)
    gv = D.Volume(0.05, 0.3, 10.0, nb, 17, 512, max_points=0, max_candidates=nb, state16=False)
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    f = f.astype(np.float32)
    f[:, 7] = 0.0       # zeros count as positive
    gv.load_fused(to_dev(f), to_dev(w.astype(np.float32)))
    st = gv.regularize(D.reg_params(LAM, iters=0, init=D.DN_INIT_GIVEN), u0=to_dev(f))
    c, nbr = host(gv.extract(D.DN_X_COORDS)), host(gv.extract(D.DN_X_NBR))
    u = f.astype(np.float64)
    pts = host(gv.extract(D.DN_X_SURFACE))
    ref = oracle.extract(c, nbr, w, u, 0.05)
    assert pts.shape == ref.shape and np.abs(pts - ref).max(initial=0.0) <= 1e-5
    E, Dd = oracle.energy(nbr, u, w, u, np.zeros((3,) + u.shape), LAM)
    assert abs(st.energy - E) <= 1e-9 * abs(E) and abs(st.dual - Dd) <= 1e-9 * abs(E)
    if nb > 20000:      # (the mesh of half of a random field's cubes is large)
        w = np.where(np.arange(nb)[:, None] % 16 == 0, w, 0.0)
        gv.load_fused(to_dev(f), to_dev(w.astype(np.float32)))
    tris = host(gv.extract(D.DN_X_MESH))
    mref, area = oracle.mesh(c, nbr, w, u, 0.05)
    assert tris.shape == mref.shape and np.abs(tris - mref).max(initial=0.0) <= 1e-5
    a, n = gv.mesh_area()
    assert n == len(mref) and abs(a - area) <= 1e-9 * max(area, 1e-30)
    print(f"{nb} blocks: {len(pts)} points, {n} triangles")
