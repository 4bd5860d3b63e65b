"""The estimator's gradient at the edges of its tiles (16 samples) and of its
workgroups (1024, beyond which each takes several tiles) against float64
autograd on the same float16 weights.  Every output is a chain of at most three
64-term float32 sums and one over the batch in short partial sums, each with
relative error below 64 x 6e-8 = 4e-6 of its terms' magnitude: 1e-5 in the norm
leaves room for cancellation between terms.
"""
import numpy as np
import pytest

from gpu_helpers import gpu_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 15, 16, 17, 250, 1024, 16383, 16400, 40001])
def test_gradient_matches_float64(batch):
    import torch
    from paper_1204_2280_amd import estimator, mibh
    gpu_context(16)
    print(f"[gpu] gradient, batch {batch}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(batch)
    rows = 5000
    _, w16 = estimator.init_weights(torch.device("cuda", 0), 3)
    w16[512:576] = 0.1  # biases that matter
    w16[4672:4736] = -0.05
    x = torch.rand((rows, 8), generator=g, device="cuda")
    t = 9.0 + 3.0 * x[:, 0] + torch.randn(rows, generator=g, device="cuda")
    idx = torch.randint(0, rows, (batch,), generator=g, device="cuda", dtype=torch.int32)
    grad, loss = mibh.mlp_gradient(w16, x, t, idx)
    again, loss2 = mibh.mlp_gradient(w16, x, t, idx)
    assert torch.equal(grad, again) and torch.equal(loss, loss2)
    w = w16.double().requires_grad_(True)
    X, T = x[idx.long()].double(), t[idx.long()].double()
    W1, b1, W2 = w[:512].reshape(64, 8), w[512:576], w[576:4672].reshape(64, 64)
    b2, w3, b3 = w[4672:4736], w[4736:4800], w[4800]
    y = torch.relu(torch.relu(X @ W1.T + b1) @ W2.T + b2) @ w3 + b3
    ref = ((y - T) ** 2).mean()
    (gref,) = torch.autograd.grad(ref, w)
    for a, b in ((0, 512), (512, 576), (576, 4672), (4672, 4736), (4736, 4800), (4800, 4801)):
        err = torch.linalg.vector_norm(grad[a:b].double() - gref[a:b]) / torch.linalg.vector_norm(gref[a:b])
        assert float(err) <= 1e-5, (a, b, float(err))
    assert abs(float(loss[0]) - ref.item()) <= 1e-5 * ref.item()
