"""Edges of the kernels' tilings and of the rules that choose between them:
remainders, the smallest and largest sizes of a range, and alignment."""
import numpy as np
import pytest

import latgen
from oracle import deflation as DF
from oracle import learned as L
from oracle import wilson as W
from tests.gpu_helpers import M_W, banner, make_lattice, nk, to_dev, to_host, torch_cuda

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


@pytest.mark.parametrize("p", [4, 15, 16, 17, 32, 33, 48, 65, 81, 97, 112, 113, 128])
@pytest.mark.parametrize("mu", [0.0, 0.3])
def test_eigenpairs_block_sizes(p, mu):
    """Blocks around the 16- and 32-vector tiles of the Gram and rotation
    kernels, up to the largest, on 2x2x4x4: the three eigenvalues nearest the
    imaginary axis against the dense eigen-decomposition, and the residuals of
    right and left vectors with the oracle's operator (tolerances of the
    solver's own tests)."""
    torch = torch_cuda()
    b = nk()
    dims, m = (2, 2, 4, 4), 3
    n = 12 * 64
    banner(f"eigenpairs p={p} mu={mu}")
    lat, u = make_lattice(dims, 0.8, seed=0)
    v0 = to_dev(latgen.random_sources(dims, p, 11))
    r = torch.empty(m * n, dtype=torch.complex128, device="cuda")
    left = torch.empty_like(r)
    if mu == 0.0:
        lam, _, resid, rc = b.nk_eig_hermitian_device(lat.h, M_W, m, p, 20, 1e-11, 400, v0, r)
        left.copy_(r)
    else:
        lam, _, resid, rc = b.nk_eig_critical_device(lat.h, M_W, mu, m, p, 20, 1e-11, 400, v0, r, left)
    assert rc == 0
    ld, _, _ = DF.critical_eigenpairs(W.dense_matrix(u, M_W, mu), m, mu == 0.0)
    assert np.max(np.abs(np.sort_complex(lam) - np.sort_complex(ld))) < 1e-10
    R, Lv = to_host(r).reshape(m, n), to_host(left).reshape(m, n)
    assert np.linalg.norm(Lv.conj() @ R.T - np.eye(m)) < 1e-10
    for i in range(m):
        f = lambda v, s: W.a_apply(u, v.reshape(4, 4, 2, 2, 4, 3), M_W, s).reshape(-1)  # noqa: E731
        assert np.linalg.norm(f(R[i], mu) - lam[i] * R[i]) < 2e-10
        assert np.linalg.norm(f(Lv[i], -mu) - np.conj(lam[i]) * Lv[i]) < 2e-10 * np.linalg.norm(Lv[i])
    lat.close()
