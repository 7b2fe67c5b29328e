"""The forward pass beyond one tile per compute unit (workgroups loop over
tiles): every tile's output is what the tile gives in a call of its own, and
the last ones agree with the oracle."""
import numpy as np
import pytest

from gpu_common import dn, host, net_forward_checks, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 257, 600])
def test_a_large_batch_equals_its_parts(n):
    D = dn()
    import torch
    rng = np.random.default_rng(n)
    prm = rng.normal(0, 0.15, D.NET_PARAMS)
    tiles = rng.normal(0, 0.6, (n, 2, 10, 10, 10))
    p, t = to_dev(prm, torch.float32), to_dev(tiles, torch.float32)
    out = torch.full((n, 10, 10, 10), float("nan"), device="cuda")
    D.net_forward(t, p, out)
    part = torch.empty((32, 10, 10, 10), device="cuda")
    for i in range(0, n, 32):
        m = min(32, n - i)
        D.net_forward_static(t[i:i + m].contiguous(), p, part[:m])
        assert torch.equal(part[:m], out[i:i + m]), i
    net_forward_checks(host(out[-3:]).astype(np.float64), tiles[-3:], prm, f"last of {n}")
