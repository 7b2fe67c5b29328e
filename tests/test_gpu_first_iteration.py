"""A solve from zero takes its first iteration without the state in memory:
the same bits as the solve that is given zeros, which takes the general
kernels throughout, in every storage, data term and step rule, after buffers
that held another state, and for sub-maps solved together."""
import numpy as np
import pytest

import scenes
from gpu_common import LAM, dn, state_of, to_dev

pytestmark = pytest.mark.gpu


def _volume(D, nb, extent, seed=5):
    coords, f, w = scenes.random_block_field(nb, seed, extent=extent, omega_frac=0.7)
    gv = D.Volume(0.1, 0.3, 10.0, nb, 12, 256, max_points=0, max_candidates=max(nb, 64))
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    gv.load_fused(to_dev(f.astype(np.float32)), to_dev(w.astype(np.float32)))
    return gv


@pytest.mark.parametrize("nb,extent", [(1, 1), (3, 2), (259, 7)])
@pytest.mark.parametrize("storage,refine", [("DN_F32", 50), ("DN_F16", 50), ("DN_BF16", 2), ("DN_BF16", 1)])
@pytest.mark.parametrize("data,gamma", [("DN_DATA_L2", 0.0), ("DN_DATA_L2", 0.5), ("DN_DATA_L1", 0.0)])
def test_from_zero_equals_given_zeros(nb, extent, storage, refine, data, gamma):
    import torch
    D = dn()
    gv = _volume(D, nb, extent)
    u0 = torch.zeros((nb, 512), device="cuda")
    p0 = torch.zeros((3, nb, 512), device="cuda")
    kw = dict(storage=getattr(D, storage), refine_every=refine, data_term=getattr(D, data), gamma=gamma)
    for iters in (0, 1, 2, 5):
        for kernel in (D.DN_K_FUSED, D.DN_K_AUTO):
            st = gv.regularize(D.reg_params(LAM, iters=iters, kernel=kernel, **kw))
            zero = state_of(D, gv)
            given = gv.regularize(D.reg_params(LAM, iters=iters, kernel=D.DN_K_FUSED, init=D.DN_INIT_GIVEN, **kw),
                                  u0, p0)
            for a, b in zip(zero, state_of(D, gv)):
                np.testing.assert_array_equal(a, b)
            assert (st.energy, st.dual, st.iters_run) == (given.energy, given.dual, given.iters_run)
        # another state in the buffers before the next solve
        gv.regularize(D.reg_params(LAM, iters=3, init=D.DN_INIT_GIVEN), u0 + 0.5, p0 + 0.25)


@pytest.mark.parametrize("gamma", [0.0, 0.5])
@pytest.mark.parametrize("kernel", ["DN_K_AUTO", "DN_K_FUSED", "DN_K_FUSED256"])
def test_batch_from_zero(gamma, kernel):
    D = dn()
    sizes = [(1, 1), (65, 5), (259, 7)]
    vols = [_volume(D, nb, extent, seed=nb) for nb, extent in sizes]
    for iters in (1, 2, 6):
        st = D.regularize_batch(vols, D.reg_params(LAM, iters=iters, kernel=getattr(D, kernel), gamma=gamma))
        for (nb, extent), gv, s in zip(sizes, vols, st):
            one = _volume(D, nb, extent, seed=nb)
            ref = one.regularize(D.reg_params(LAM, iters=iters, kernel=D.DN_K_FUSED, gamma=gamma))
            for a, b in zip(state_of(D, gv), state_of(D, one)):
                np.testing.assert_array_equal(a, b)
            assert (s.energy, s.dual) == (ref.energy, ref.dual)
            one.close()
