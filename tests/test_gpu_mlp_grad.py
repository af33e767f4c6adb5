"""The gradient of the learned indicator's network at batch sizes around the
kernel's tiles: within one pass of 64 samples, at its edges, around the 256 blocks
of one pass each, and with blocks that make several passes; for device inputs at any
4-byte alignment.

Reference: the oracle's FP64 gradient at the BF16 weights.  Every entry of the
gradient is a chain of at most 16 + 64 + 64 products forward, 64 backward, 64 per
pass over the samples, three passes at these sizes, and 32 partial sums: some 400
roundings of 2^-24, so 400 2^-24 = 2.4e-5 of the norm bounds the error if they all had
the same sign; the loss has 64 + 32 more on the forward ones, 1.5e-5."""
import numpy as np
import pytest

from oracle import mlp as MLP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 31, 33, 64, 65, 128, 8192, 16384, 16385, 40001])
def test_gradient_by_batch_size(B):
    import paper_2607_06045_amd as P
    import torch
    s = P.Solver(3)
    w = MLP.init(B % 17)
    s.mlp_set_weights(w)
    rng = np.random.default_rng(B)
    x = rng.uniform(0, 1, (B, 16)).astype(np.float32)
    t = rng.uniform(0, 0.5, B).astype(np.float32)
    loss_ref, g_ref = MLP.loss_and_grad(w, x.astype(np.float64), t.astype(np.float64))
    g, loss = s.mlp_grad(x, t)
    rel = np.linalg.norm(g - g_ref) / np.linalg.norm(g_ref)
    print(f"grad B={B}: rel {rel:.2e} loss {abs(loss - loss_ref) / loss_ref:.2e}", flush=True)
    assert rel < 2.4e-5 and abs(loss - loss_ref) <= 1.5e-5 * loss_ref
    flat = torch.zeros(16 * B + 4, dtype=torch.float32, device="cuda")
    td = torch.from_numpy(t).cuda()
    for off in (0, 1):
        xd = flat[off:off + 16 * B].view(B, 16)
        xd.copy_(torch.from_numpy(x))
        gd, ld = s.mlp_grad(xd, td)
        assert np.array_equal(gd.cpu().numpy(), g) and ld == loss
