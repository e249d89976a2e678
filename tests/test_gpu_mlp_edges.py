"""The proposal network's forward and backward passes at batch sizes around
their blocks (16 samples, 32 in the weight gradient) against
oracle/mlp_ref.py."""
import numpy as np
import pytest

from oracle import mlp_ref as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 200, 1025])
def test_batch_edges(n):
    import torch
    from paper_2502_20072_amd import _binding as B
    rng = np.random.default_rng(n)

    def f32(a):
        return np.asarray(a, dtype=np.float32).astype(np.float64)

    def t(a):
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda:0")
    flat = f32(rng.normal(0, 0.15, R.NPARAM))
    X, Y = f32(rng.normal(size=(2 * n + 20, R.IN))), f32(rng.normal(size=n))
    # no hidden unit so near zero that FP32 rounding (about 1e-6) could switch it
    _, (_, z1, _, z2, _) = R.forward(flat, X)
    X = X[np.minimum(np.abs(z1).min(1), np.abs(z2).min(1)) > 5e-6][:n]
    assert len(X) == n
    st = torch.cuda.current_stream().cuda_stream
    P, Xd, Yd = t(flat), t(X), t(Y)
    ws = torch.empty(B.sisso_mlp_workspace_bytes(n), dtype=torch.uint8, device="cuda:0")
    out = torch.empty(n, dtype=torch.float32, device="cuda:0")
    grad = torch.full((R.NPARAM,), float("nan"), dtype=torch.float32, device="cuda:0")
    loss = torch.empty(1, dtype=torch.float32, device="cuda:0")
    B.sisso_mlp_forward(P, Xd, out, ws, st)
    B.sisso_mlp_backward(P, Xd, Yd, grad, loss, ws, st)
    ref_out, _ = R.forward(flat, X)
    ref_loss, ref_g = R.loss_and_grad(flat, X, Y)
    np.testing.assert_allclose(out.cpu().numpy(), ref_out, rtol=0, atol=2e-5 * np.max(np.abs(ref_out)))
    assert abs(loss.item() - ref_loss) <= 1e-4 * ref_loss
    np.testing.assert_allclose(grad.cpu().numpy(), ref_g, rtol=0, atol=2e-5 * np.max(np.abs(ref_g)))
