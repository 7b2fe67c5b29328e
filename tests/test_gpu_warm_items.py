"""The warm start's workgroups loop over (block, axis) items, 512 at a time on
256 compute units: sparse block sets with fewer, as many and more items,
against the oracle, both modes."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_common import dn, dual_warm_start_checks, host, net_forward_checks, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,extent", [(1, 1), (40, 6), (171, 7), (513, 10)])
def test_sparse_sets_of_every_size(nb, extent):
    D = dn()
    import torch
    coords, f, w = scenes.random_block_field(nb, 3, extent=extent, omega_frac=0.8)
    gv = D.Volume(0.1, 0.3, 10.0, nb, 12, 256, max_points=0, max_candidates=max(nb, 64))
    gv.insert_blocks(to_dev(coords.astype(np.int32)), keep_order=True)
    gv.load_fused(to_dev(f.astype(np.float32)), to_dev(w.astype(np.float32)))
    prm = np.random.default_rng(nb).normal(0, 0.1, D.NET_PARAMS)
    t = to_dev(prm, torch.float32)
    u0 = torch.full((nb, 512), float("nan"), device="cuda")
    p0 = torch.full((3, nb, 512), float("nan"), device="cuda")
    gv.net_warm_start(t, u0, p0, mode=D.DN_WARM_DUAL)
    dual = host(p0).astype(np.float64)
    primal = torch.full((nb, 512), float("nan"), device="cuda")
    gv.net_warm_start(t, primal, None, mode=D.DN_WARM_PRIMAL, delta=0.1)
    primal = host(primal).astype(np.float64)
    nbr, em = host(gv.extract(D.DN_X_NBR)), host(gv.extract(D.DN_X_EMASK))
    f = f.astype(np.float32).astype(np.float64)
    # the first, the last and some between (every workgroup's first and later items)
    some = np.unique(np.concatenate([np.arange(min(nb, 4)), np.linspace(0, nb - 1, 12).astype(int),
                                     np.arange(max(nb - 4, 0), nb)])).astype(np.int32)
    dual_warm_start_checks(dual[:, some], nbr, f, w, some, em[some], prm, f"dual, {nb} blocks")
    assert np.isfinite(dual).all() and np.isfinite(primal).all()
    tiles = oracle.net_gather(nbr, f, w, some)
    r64 = oracle.net_forward(tiles, prm, gate=0)[:, 1:9, 1:9, 1:9].reshape(-1, 512)
    keep = np.zeros((len(some), 10, 10, 10), bool)
    keep[:, 1:9, 1:9, 1:9] = ((w[some] > 0) & (np.abs(primal[some]) < 1) &
                              (np.abs(f[some] + r64) < 1)).reshape(-1, 8, 8, 8)
    r_dev = np.zeros((len(some), 10, 10, 10))
    r_dev[:, 1:9, 1:9, 1:9] = (primal[some] - f[some]).reshape(-1, 8, 8, 8)
    net_forward_checks(r_dev, tiles, prm, f"primal, {nb} blocks", region=lambda a: a[keep])
    assert (primal[w == 0] == 0).all()
