"""Gradient kernel of the threshold model at the edges of its chunks of 32
samples and of its grid of 256 workgroups, against float64 autograd."""
import numpy as np
import pytest
import torch

import paper_1908_09378_amd as pkg
from paper_1908_09378_amd import learn

pytestmark = pytest.mark.gpu


def reference(X, Y, blob):
    b = blob.double()
    p = b[:pkg.MLP_PARAMS].float().to(torch.bfloat16).double().requires_grad_(True)
    mu, sd = b[pkg.MLP_PARAMS:pkg.MLP_PARAMS + 8], b[pkg.MLP_PARAMS + 8:pkg.MLP_PARAMS + 16]
    w1, b1, w2, b2, w3, b3 = torch.split(p, [512, 64, 4096, 64, 64, 1])
    h = torch.nn.functional.gelu((X.double() - mu) / sd @ w1.view(8, 64) + b1)
    h = torch.nn.functional.gelu(h @ w2.view(64, 64) + b2)
    loss = ((h @ w3 + b3 - Y.double()) ** 2).mean()
    return torch.autograd.grad(loss, p)[0], loss.detach()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 65, 1000, 32 * 256, 32 * 256 + 5, 65536])
def test_gradient_at_chunk_and_grid_edges(n):
    g = torch.Generator().manual_seed(n)
    X = (torch.randn(n, 8, generator=g) * 2 + 1).float()
    Y = torch.rand(n, generator=g).float() * 5
    blob = torch.from_numpy(learn.init_blob(n))
    blob[:pkg.MLP_PARAMS] += 0.05 * torch.randn(pkg.MLP_PARAMS, generator=g)
    blob[pkg.MLP_PARAMS:pkg.MLP_PARAMS + 8] = 1.0
    blob[pkg.MLP_PARAMS + 8:pkg.MLP_PARAMS + 16] = 2.0
    ref, rloss = reference(X, Y, blob)
    grad = torch.empty(pkg.MLP_PARAMS, device="cuda")
    loss = torch.empty(1, device="cuda")
    pkg.mlp_grad(X.cuda(), Y.cuda(), blob.cuda(), grad, loss)
    # float32 products and sums: each term carries a few roundings of the
    # forward and backward chains (64-term dot products, erff, expf), and the
    # sums are trees of at most 256 + 8 levels of 32 terms
    tol = 2e-5 * float(ref.abs().max())
    assert float((grad.cpu().double() - ref).abs().max()) <= tol
    assert abs(float(loss) - float(rloss)) <= 2e-5 * float(rloss)


def test_training_step_follows_the_gradient():
    """One Adam step moves every parameter by lr * g / (|g| + eps) (then
    bfloat16 rounding), so the step's sign is the gradient's."""
    g = torch.Generator().manual_seed(5)
    X = (torch.randn(100, 8, generator=g) * 2 + 1).float().cuda()
    Y = (torch.rand(100, generator=g) * 5).float().cuda()
    start = torch.from_numpy(learn.init_blob(3)).cuda()
    blob = start.clone()
    grad, loss = torch.empty(pkg.MLP_PARAMS, device="cuda"), torch.empty(1, device="cuda")
    pkg.mlp_grad(X, Y, start, grad, loss)
    lt = pkg.mlp_train(X, Y, blob, 100, 1, 0.125)
    want = (start[:pkg.MLP_PARAMS] - 0.125 * grad / (grad.abs() + 1e-8)).to(torch.bfloat16).float()
    assert np.allclose(lt[0], float(loss), rtol=1e-6)
    # equal up to one bfloat16 step where the float32 values straddle a tie
    diff = (blob[:pkg.MLP_PARAMS] - want).abs()
    assert bool((diff <= 2.0 ** -8 * want.abs() + 1e-6).all())
