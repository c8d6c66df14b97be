"""The scorer's forward pass with an output where an earlier layer's rows lie
(scores over the features or over h1, h2 over the features): the same values
as with buffers apart, whatever order the tiles run in."""
import numpy as np
import pytest

from oracle import mlp
from paper_1805_00475_amd import tn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 17, 3000, 5000])
@pytest.mark.parametrize("share", ["y=x", "y=h1", "h2=x", "y end of x", "h2=h1"])
def test_shared_outputs(n, share):
    import torch
    print("[gpu case] mlp forward", n, share, flush=True)
    r = np.random.default_rng(n)
    X = torch.from_numpy(r.normal(0, 1, (n, mlp.F)).astype(np.float32)).cuda()
    P = torch.from_numpy(mlp.init_params(n).astype(np.float32)).cuda()
    f = dict(dtype=torch.float32, device="cuda")
    h1, h2, y = torch.empty(n, mlp.H, **f), torch.empty(n, mlp.H, **f), torch.empty(n, **f)
    tn.mlp_forward(P, X, h1, h2, y)
    big = torch.zeros(n, mlp.H, **f)
    g1, g2, gy, x = torch.zeros(n, mlp.H, **f), torch.zeros(n, mlp.H, **f), torch.zeros(n, **f), X.clone()
    if share == "y=x":
        gy = x.view(-1)[:n]
    elif share == "y end of x":
        gy = x.view(-1)[-n:]
    elif share == "y=h1":
        gy = g1.view(-1)[:n]
    elif share == "h2=h1":
        g2 = g1
    else:
        # the features at the end of h2's buffer
        big.view(-1)[-n * mlp.F:] = x.view(-1)
        x = big.view(-1)[-n * mlp.F:].view(n, mlp.F)
        g2 = big
    tn.mlp_forward(P, x, g1, g2, gy)
    torch.cuda.synchronize()
    assert torch.equal(gy, y)
    assert share == "y=h1" or torch.equal(g2, h2)
    assert share in ("y=h1", "h2=h1") or torch.equal(g1, h1)
