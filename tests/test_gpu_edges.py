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


@pytest.mark.parametrize("B", [1, 17, 65, 2048])
def test_mlp_forward_is_double_up_to_storage(B):
    """The forward pass computes in FP64 and rounds to FP32 where y and the
    activations are stored: 2^-24 of each, 6e-8, and no more of their norms
    (sums in FP32 are off by 2e-7)."""
    torch = torch_cuda()
    b = nk()
    rng = np.random.default_rng(B)
    p = latgen.mlp_init(B).astype(np.float32)
    p[:L.NTRAIN] += (0.1 * rng.standard_normal(L.NTRAIN)).astype(np.float32)
    f = rng.standard_normal((B, L.NIN)).astype(np.float32)
    banner(f"mlp forward in FP64, batch {B}")
    y = torch.zeros((B, L.T), dtype=torch.float32, device="cuda")
    act = torch.zeros((B, 3, L.NH), dtype=torch.float32, device="cuda")
    b.nk_mlp_forward_device(torch.from_numpy(p).cuda(), torch.from_numpy(f).cuda(), y, act)
    ref, acts = L.forward(p.astype(np.float64), f.astype(np.float64))
    off = lambda got, want: np.linalg.norm(got - want) / np.linalg.norm(want)  # noqa: E731
    assert off(y.cpu().numpy(), ref) < 6e-8
    for i in range(3):
        assert off(act.cpu().numpy()[:, i], acts[1 + i]) < 6e-8


def test_spectral_loss_sizes():
    """Spectra at the edges of the kernel's slots (256, 512 and 1024
    eigenvalues) and of a wave, and an empty one, in one batch against the
    oracle.  The arithmetic is FP64 (sums of n terms, conditions below 1e4:
    1e-10), the results FP32: 6e-8 of each, with a margin."""
    torch = torch_cuda()
    b = nk()
    rng = np.random.default_rng(9)
    sizes = [1, 64, 65, 255, 256, 257, 0, 320, 511, 512, 513, 1024]
    lams = [(rng.uniform(0.3, 6.0, n) * rng.choice([-1.0, 1.0], n) + 0.2j * rng.standard_normal(n)) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    y = (0.4 * rng.standard_normal((len(sizes), L.T))).astype(np.float32)
    banner(f"spectral loss, spectra of {sizes}")
    loss = torch.full((len(sizes),), 7.0, dtype=torch.float32, device="cuda")
    dy = torch.full((len(sizes), L.T), 7.0, dtype=torch.float32, device="cuda")
    b.nk_rh_spectral_loss_device(torch.from_numpy(off).cuda(), torch.from_numpy(np.concatenate(lams)).cuda(),
                                 torch.from_numpy(y).cuda(), 0.25, loss, dy)
    for i, lam in enumerate(lams):
        lr, gr = L.spectral_loss(lam, y[i].astype(np.float64)) if len(lam) else (0.0, np.zeros(L.T))
        assert abs(loss[i].item() - lr) <= 1e-6 * max(1.0, abs(lr)), sizes[i]
        assert np.allclose(dy[i].cpu().numpy(), 0.25 * gr, rtol=1e-6, atol=1e-8), sizes[i]


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


def _tridiag(kind, n, seed):
    """Tridiagonal matrices (diagonal, super-, sub-diagonal) away from the imaginary axis."""
    rng = np.random.default_rng([seed, n])
    c = lambda: rng.standard_normal(n) + 1j * rng.standard_normal(n)  # noqa: E731
    if kind == "zerodiag":  # zero pivots at every other step; spectrum +-(1 +- 0.3)
        b = np.where(np.arange(n) % 2 == 0, 1.3, 0.3) + 0j
        return np.zeros(n, np.complex128), b, b.copy()
    if kind == "real":  # Hermitian, two intervals
        a = np.where(np.arange(n) % 2 == 0, 2.0, -2.0) + 0.3 * rng.standard_normal(n)
        b = 0.8 + 0.2 * rng.random(n)
        return a + 0j, b + 0j, b + 0j
    if kind == "complex":
        a = np.where(rng.random(n) < 0.5, 3.0, -3.0) + 0.3 * c()
        return a, 0.6 * c(), 0.6 * c()
    a, b, d = _tridiag("real", n, seed)  # slow: an eigenvalue 1e-4 of the others' size in an uncoupled corner
    a[-1] = 2e-4
    if n > 1:
        b[n - 2] = d[n - 2] = 0.0
    return a, b, d


def _dense(a, b, d):
    return np.diag(a) + np.diag(b[:-1], 1) + np.diag(d[:-1], -1)


@pytest.mark.parametrize("n", [1, 2, 3, 5, 16, 31, 63, 64, 65, 127, 128, 129, 192, 193, 255, 257, 320, 511])
@pytest.mark.parametrize("kind", ["real", "complex", "zerodiag", "slow"])
def test_tridiagonal_sign_orders(kind, n):
    """sgn(T) e_1 of tridiagonal T over the edges of the 64-column and 128-row
    tiles and of the rule between 4 and 16 poles at a time, unscaled and with
    determinant scaling: against the oracle's Roberts-Higham iteration with
    explicit inverses (1e-10, the tolerance of the dense iteration's tests) and
    the spectral sign, with the iteration count to +-1.  "zerodiag" meets exact
    zero pivots, "slow" goes past the steps taken in closed form."""
    from oracle import dense as D
    from oracle import rh as R
    if kind == "zerodiag" and n % 2:
        n += 1  # an odd one is singular
    b = nk()
    a, be, de = _tridiag(kind, n, 5)
    T = _dense(a, be, de)
    banner(f"tridiagonal sign {kind} n={n}")
    so, ito, _ = R.roberts_higham(T)
    ref = D.sign_spectral(T, hermitian=False)
    for scaling in (b.NK_RH_NONE, b.NK_RH_DET):
        z, info, rc = b.nk_small_sign(n, 0, kind != "complex", a, be, de, b.nk_sign_params_default(rh_scaling=scaling))
        assert rc == 0
        assert np.linalg.norm(z - so[:, 0]) < 1e-10 and np.linalg.norm(z - ref[:, 0]) < 1e-9
        assert info.rh_residual < 1e-9
        if scaling == b.NK_RH_NONE:
            assert abs(info.rh_iters - ito) <= 1
        else:
            _, itd, _ = R.roberts_higham(T, scale=R.determinant_scale)
            assert abs(info.rh_iters - itd) <= 1


@pytest.mark.parametrize("n", [6, 60, 128, 130, 300])
@pytest.mark.parametrize("maxit", [1, 2, 3, 4, 5, 7, 9, 10, 11])
@pytest.mark.parametrize("det", [False, True])
def test_tridiagonal_sign_capped(n, maxit, det):
    """The iterate after every possible cap equals the oracle's (the steps taken
    in closed form, and those after them, are Eq. (4)'s)."""
    from oracle import rh as R
    b = nk()
    a, be, de = _tridiag("slow", n, 9)
    T = _dense(a, be, de)
    S, it, _ = R.roberts_higham(T, maxit=maxit, scale=R.determinant_scale if det else None)
    banner(f"tridiagonal sign n={n} maxit={maxit} det={det}")
    p = b.nk_sign_params_default(rh_maxit=maxit, rh_scaling=b.NK_RH_DET if det else b.NK_RH_NONE)
    z, info, rc = b.nk_small_sign(n, 0, True, a, be, de, p)
    assert info.rh_iters == it
    assert rc == (b.NK_WARN_NOTCONV if it == maxit else 0) or it == maxit
    assert np.linalg.norm(z - S[:, 0]) <= 1e-11 * max(1.0, np.linalg.norm(S[:, 0]))


@pytest.mark.parametrize("n", [1, 3, 97, 200])
def test_tridiagonal_sign_singular(n):
    """A singular matrix, and one with the eigenvalue i (whose first iterate is
    singular), are reported as by the dense iteration."""
    b = nk()
    for last in (0.0, 1j):
        a, be, de = _tridiag("slow", n, 3)
        a[-1] = last
        banner(f"tridiagonal sign n={n} with eigenvalue {last}")
        _, _, rc = b.nk_small_sign(n, 0, False, a, be, de)
        assert rc == b.NK_WARN_NOTCONV
        assert "singular" in b.nk_last_error()


def test_tridiagonal_sign_nan_is_reported():
    b = nk()
    a, be, de = _tridiag("real", 70, 4)
    a[30] = np.nan
    _, _, rc = b.nk_small_sign(70, 0, True, a, be, de)
    assert rc == b.NK_WARN_NOTCONV


def _two_sided(B, ell):
    """Diagonal, super- and sub-diagonal of H_ell of K_ell(B, e_1), two-sided, each projection twice."""
    k = len(B)
    V, Wd = np.zeros((k, ell), complex), np.zeros((k, ell), complex)
    V[0, 0] = Wd[0, 0] = 1.0
    a, be, de = np.zeros(ell, complex), np.zeros(ell - 1, complex), np.zeros(ell - 1, complex)
    for i in range(ell):
        u, q = B @ V[:, i], B.conj().T @ Wd[:, i]
        a[i] = np.vdot(Wd[:, i], u)
        for _ in range(2):
            u, q = u - V[:, :i + 1] @ (Wd[:, :i + 1].conj().T @ u), q - Wd[:, :i + 1] @ (V[:, :i + 1].conj().T @ q)
        if i + 1 < ell:
            s = np.vdot(q, u)
            de[i] = np.sqrt(abs(s))
            be[i] = s / de[i]
            V[:, i + 1], Wd[:, i + 1] = u / de[i], q / np.conj(be[i])
    return a, be, de


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 17, 959, 960, 961, 1365, 1366])
@pytest.mark.parametrize("diag", [0.3, 3.0])
@pytest.mark.parametrize("e", [0, 230, -230])
def test_inner_projection_of_every_elimination(k, diag, e):
    """H_ell around the sizes at which the elimination of H_k changes its
    storage, with rows exchanged (a small diagonal) and not, and with pivots
    beyond the range of its unscaled reciprocal (H_k 2^230: B = H_k to the last
    bit, 2^-230: B = H_k^{-1}).  Five steps in FP64, condition below 100: 1e-10."""
    b = nk()
    rng = np.random.default_rng(1000 + k)
    c = lambda n: rng.standard_normal(n) + 1j * rng.standard_normal(n)
    al, be, de = diag * np.exp(0.3j * rng.standard_normal(k)) + 0.05 * c(k), 1.0 + 0.1 * c(k), 1.1 + 0.1 * c(k)
    if diag < 1.0:  # weakly coupled pairs
        be[1::2], de[1::2] = 0.2 * be[1::2], 0.2 * de[1::2]
    H = np.diag(al) + np.diag(be[:k - 1], 1) + np.diag(de[:k - 1], -1)
    assert np.linalg.cond(H) < 100
    ell = min(5, k - 1) if k > 1 else 1
    B = H + np.linalg.inv(H) if e == 0 else H if e > 0 else np.linalg.inv(H)
    ref = _two_sided(B, ell)
    banner(f"inner projection k={k} diagonal {diag} scale 2^{e}")
    f = 2.0 ** e
    got = b.nk_inner_matrix(k, ell, False, f * al, f * be, f * de)
    assert got[3] == ell and got[4] == 0
    g = 2.0 ** -abs(e)
    for x, y in zip(got[:3], ref):
        x = g * x[:len(y)]
        assert np.linalg.norm(x - y) <= 1e-10 * max(1.0, np.linalg.norm(ref[0]))


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 2), (16, 4, 2, 2), (6, 4, 2, 10), (8, 8, 4, 6)])
@pytest.mark.parametrize("shift", [None, 5, 12, -7, 0.5, 1.0, -1.0])
def test_operator_on_apart_and_overlapping_vectors(dims, shift):
    """Canonical vectors with x and y apart (one launch), and y anywhere over x:
    then each x is read as the outputs before it left it.  Sites below, at and
    above a wave's 64; a fixed sum of at most 8 x 2 x 9 products: 1e-13."""
    b = nk()
    torch = torch_cuda()
    lat, u = make_lattice(dims, 0.8, seed=3)
    nrhs = 3
    x = latgen.random_sources(dims, nrhs, 4).reshape(nrhs, -1)
    n = x.shape[1]
    banner(f"operator dims={dims} shift={shift}")
    buf = np.zeros(6 * n, complex)
    ix = n if shift is not None and shift < 0 else 0
    buf[ix:ix + 3 * n] = x.reshape(-1)
    iy = 3 * n if shift is None else ix + (shift if isinstance(shift, int) else int(shift * n))
    ref = buf.copy()
    for r in range(nrhs):
        src = ref[ix + r * n:ix + (r + 1) * n].reshape(latgen.random_sources(dims, 1, 0)[0].shape)
        ref[iy + r * n:iy + (r + 1) * n] = np.asarray(W.dw_apply(u, src.copy(), M_W, 0.3, g5=True)).reshape(-1)
    for call in (b.nk_apply_dw_device, b.nk_apply_dw_noalloc_device):
        t = torch.from_numpy(buf.copy()).cuda()
        call(lat.h, M_W, 0.3, True, t[ix:ix + 3 * n], t[iy:iy + 3 * n], nrhs)
        got = to_host(t)
        assert np.linalg.norm(got - ref) <= 1e-13 * np.linalg.norm(ref)
    lat.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (4, 2, 6, 2), (16, 4, 2, 2), (6, 4, 2, 10)])
def test_spinor_layouts_are_inverse(dims):
    """Packing is a permutation (every entry once) and unpacking undoes it, on
    site counts below, at and above a workgroup's 64."""
    b = nk()
    torch = torch_cuda()
    lat, _ = make_lattice(dims, 0.8, seed=3)
    n = 12 * int(np.prod(dims))
    x = torch.arange(2 * n, dtype=torch.float64, device="cuda") + 0.5j
    xp, back = torch.zeros_like(x), torch.zeros_like(x)
    b.nk_spinor_pack_device(lat.h, x, xp, 2)
    b.nk_spinor_unpack_device(lat.h, xp, back, 2)
    assert torch.equal(back, x)
    for r in range(2):
        assert torch.equal(torch.sort(xp[r * n:(r + 1) * n].real).values, x[r * n:(r + 1) * n].real)
    lat.close()


@pytest.mark.parametrize("dims", [(16, 16, 28, 28), (24, 24, 18, 20)])
def test_pair_on_both_sides_of_the_cache_size(dims):
    """The fused pair against two single applications where its links and
    fields just fill the 256 MB cache (200704 sites are above 199728, 207360
    further; the smaller lattices of the other tests are below): the same sum of
    8 x 2 x 3 products per entry, 1e-14."""
    b = nk()
    torch = torch_cuda()
    lat, _ = make_lattice(dims, 0.8, seed=3)
    n = 12 * int(np.prod(dims))
    banner(f"pair dims={dims}")
    gen = torch.Generator(device="cuda").manual_seed(5)
    v, w = (torch.randn(n, dtype=torch.complex128, device="cuda", generator=gen) for _ in range(2))
    av, aw, rv, rw = (torch.zeros_like(v) for _ in range(4))
    b.nk_apply_pair_packed_device(lat.h, M_W, 0.3, v, w, av, aw)
    b.nk_apply_dw_packed_device(lat.h, M_W, 0.3, True, v, rv)
    b.nk_apply_dw_packed_device(lat.h, M_W, -0.3, True, w, rw)
    for got, ref in ((av, rv), (aw, rw)):
        assert torch.linalg.vector_norm(got - ref) <= 1e-14 * torch.linalg.vector_norm(ref)
    lat.close()
