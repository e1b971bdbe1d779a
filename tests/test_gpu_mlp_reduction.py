"""The training gradient's sum over workgroup partials, at the row counts
where the summing kernel's split changes (a row is 256 samples): one row,
fewer rows than row classes, one more, more than a lane's loads in flight,
and the largest, where waves take more than one tile."""
import numpy as np
import pytest

import oracle
from test_gpu_mlp import BLOCKS, _dev, _params, _rounded_reference_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31 * 128, 32 * 128 + 1, 128 * 128 + 1, 1024 * 128 + 33,
                               31 * 256, 32 * 256 + 1, 128 * 256 + 1, 1024 * 256 + 33])
def test_gradient_at_partial_counts(lib, n):
    """Each parameter block within 1e-2 of the reference that rounds to bf16
    where the kernels do (the bound of the gradient-block test)."""
    import torch
    ctx = lib.Context(0)
    rs = np.random.default_rng(n)
    P = _params(n, 0.3)
    X = rs.uniform(0, 1, size=(n, 8)).astype(np.float32)
    Y = rs.dirichlet(np.ones(4), size=(n, 2)).reshape(n, 8).astype(np.float32)
    Cc = (rs.random(n) < 0.5).astype(np.float32)
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    grad = torch.full((oracle.MLP_NPARAM,), np.nan, dtype=torch.float32, device="cuda")
    ctx.mlp_loss_grad(_dev(P), _dev(X), _dev(Y), _dev(Cc), loss, grad)
    g = grad.cpu().numpy().astype(np.float64)
    ref = _rounded_reference_grad(P, X, Y, Cc.astype(np.float64))
    for name, sl in BLOCKS.items():
        assert np.linalg.norm(g[sl] - ref[name]) <= 1e-2 * np.linalg.norm(ref[name]) + 1e-30, name
    again = torch.zeros_like(grad)
    ctx.mlp_loss_grad(_dev(P), _dev(X), _dev(Y), _dev(Cc), loss, again)
    assert torch.equal(grad, again)
