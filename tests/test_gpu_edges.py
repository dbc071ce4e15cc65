"""Edges of the kernels' tilings and of the rules that choose between them:
remainders, the smallest and largest sizes of a range, and alignment."""
import numpy as np
import pytest

import latgen
from oracle import learned as L
from tests.gpu_helpers import banner, nk, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,shift", [(1, 0), (15, 0), (16, 1), (17, 0), (63, 0), (64, 0), (65, 1), (257, 0), (2048, 0)])
def test_mlp_batch_remainders(B, shift):
    """Forward and backward over batches around the 16 samples of a forward tile
    and the 64 of a gradient step, with the flat parameters at any 4-byte
    alignment.  FP32 sums of up to 64 terms and of B terms in groups: a relative
    rounding of a few times 1e-6 at the most, held to 2e-5."""
    torch = torch_cuda()
    b = nk()
    rng = np.random.default_rng(100 + B)
    p = latgen.mlp_init(B).astype(np.float32)
    p[:L.NTRAIN] += (0.1 * rng.standard_normal(L.NTRAIN)).astype(np.float32)
    f = rng.standard_normal((B, L.NIN)).astype(np.float32)
    dyh = rng.standard_normal((B, L.T)).astype(np.float32)
    banner(f"mlp batch {B}, parameters shifted by {shift}")
    store = torch.zeros(p.size + shift, dtype=torch.float32, device="cuda")
    P = store[shift:]
    P.copy_(torch.from_numpy(p))
    F = torch.from_numpy(f).cuda()
    y = torch.zeros((B, L.T), dtype=torch.float32, device="cuda")
    act = torch.zeros((B, 3, L.NH), dtype=torch.float32, device="cuda")
    delta = torch.zeros_like(act)
    grad = torch.full((L.NTRAIN,), 7.0, dtype=torch.float32, device="cuda")
    b.nk_mlp_forward_device(P, F, y, act)
    b.nk_mlp_backward_device(P, F, act, torch.from_numpy(dyh).cuda(), delta, grad)
    ref, acts = L.forward(p.astype(np.float64), f.astype(np.float64))
    g = L.backward(p.astype(np.float64), acts, dyh.astype(np.float64))
    off = lambda got, want: np.linalg.norm(got - want) / np.linalg.norm(want)  # noqa: E731
    assert off(y.cpu().numpy(), ref) < 2e-5
    for i in range(3):
        assert off(act.cpu().numpy()[:, i], acts[1 + i]) < 2e-5
    assert off(grad.cpu().numpy(), g) < 2e-5
