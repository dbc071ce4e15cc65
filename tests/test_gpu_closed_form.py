"""Roberts-Higham from a tridiagonal matrix in closed form, where it ends and
the iteration with explicit inverses takes over: caps, badly scaled entries,
loose tolerances, wide spectra and the workspace's bound."""
import numpy as np
import pytest

import latgen
from tests.gpu_helpers import banner, make_lattice, nk, rel, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu


def _dense(a, b, d):
    return np.diag(a) + np.diag(b[:-1], 1) + np.diag(d[:-1], -1)


def _intervals(n, seed):
    """Hermitian: diagonal +-2, off-diagonal about 0.9 (n = 1: the diagonal alone)."""
    rng = np.random.default_rng([seed, n])
    a = np.where(np.arange(n) % 2 == 0, 2.0, -2.0) + 0.1 * rng.standard_normal(n)
    b = 0.9 + 0.05 * rng.standard_normal(n)
    return a + 0j, b + 0j, b + 0j


@pytest.mark.parametrize("n,ell", [(1, 0), (6, 0), (128, 0), (130, 0), (6, 3), (130, 3)])
@pytest.mark.parametrize("maxit", [0, -1, -7])
def test_cap_below_one_takes_no_step(n, ell, maxit):
    """Under a cap of no step the iterate is the start matrix, unchanged, and
    the call warns: z = H e_1 (plain, exact), V_l H_l e_1 = B e_1 (nested: a sum of
    three terms and one inverse of condition below 10, 1e-12)."""
    b = nk()
    a, be, de = _intervals(n, 1)
    T = _dense(a, be, de)
    banner(f"cap {maxit} n={n} ell={ell}")
    for scaling in (b.NK_RH_NONE, b.NK_RH_DET, b.NK_RH_LEARNED):
        p = b.nk_sign_params_default(rh_maxit=maxit, rh_scaling=scaling)
        z, _, rc = b.nk_small_sign(n, ell, True, a, be, de, p)
        assert rc == b.NK_WARN_NOTCONV
        if ell == 0:
            assert np.array_equal(z, T[:, 0])
        else:
            assert np.linalg.norm(z - (T + np.linalg.inv(T))[:, 0]) < 1e-12


def _graded(kind, n, r):
    """The intervals above with one diagonal entry of r, one coupled pair of r,
    a coupling of r one way and 1 / r the other, or the lower half divided by r."""
    a, b, d = _intervals(n, 7)
    j = n // 3
    if kind == "diagonal":
        a[j] = r
    elif kind == "pair":
        b[j] = d[j] = r
    elif kind == "one side":
        b[j], d[j] = r, 1.0 / r
    else:
        a[n // 2:] /= r
        b[n // 2 - 1:] /= r
        d[n // 2 - 1:] /= r
    return a, b, d


@pytest.mark.parametrize("n", [6, 40, 128, 130])
@pytest.mark.parametrize("kind", ["diagonal", "pair", "one side", "rows"])
def test_badly_scaled_entries(kind, n):
    """Entries of 1e8 to 1e22 times their neighbours: up to 2^50 (1e15) in
    closed form, beyond it with explicit inverses.  The oracle's iteration is
    within 6e-16 of the same one in long double on these matrices; the
    tolerance of the capped iterates, 1e-11, is kept."""
    from oracle import rh as R
    b = nk()
    for r in (1e8, 7e9, 1e10, 1e12, 1e15, 1e17, 1e22):
        a, be, de = _graded(kind, n, r)
        T = _dense(a, be, de)
        for scaling, scale in ((b.NK_RH_NONE, None), (b.NK_RH_DET, R.determinant_scale)):
            S, it, _ = R.roberts_higham(T, maxit=200, scale=scale)
            banner(f"{kind} {r:g} n={n} scaling={scaling}")
            p = b.nk_sign_params_default(rh_scaling=scaling, rh_maxit=200)
            z, info, rc = b.nk_small_sign(n, 0, kind != "one side", a, be, de, p)
            assert rc == 0 and abs(info.rh_iters - it) <= 2, (r, scaling, info.rh_iters, it, rc)
            assert np.linalg.norm(z - S[:, 0]) <= 1e-11 * np.linalg.norm(S[:, 0]), (r, scaling)


@pytest.mark.parametrize("n,ell", [(40, 20), (130, 60)])
@pytest.mark.parametrize("r", [1e10, 1e12, 1e14])
def test_badly_scaled_inner_problem(n, ell, r):
    """Nested, with an entry of r in H_k and so in H_l (its off-diagonals then
    spread from 1 / r to r; the inner recurrence amplifies rounding by as much, so
    the entries of z are not determined): sgn(H_l) is unitary and V_l has
    orthonormal columns, |z| = 1 to the 1e-13 that the spread leaves of it, held to 1e-10."""
    b = nk()
    a, be, de = _graded("diagonal", n, r)
    banner(f"nested {n}/{ell} with an entry of {r:g}")
    for scaling in (b.NK_RH_NONE, b.NK_RH_DET):
        z, info, rc = b.nk_small_sign(n, ell, True, a, be, de, b.nk_sign_params_default(rh_scaling=scaling))
        assert rc == 0 and info.ell_used == ell
        assert abs(np.linalg.norm(z) - 1.0) < 1e-10


@pytest.mark.parametrize("n", [6, 60, 128, 130, 300])
@pytest.mark.parametrize("tol", [0.3, 1e-2, 1e-4, 2e-9, 1e-10])
def test_loose_tolerance_returns_the_iterate_it_names(n, tol):
    """With a loose tolerance the result is iterate rh_iters of Eq. (4), not a
    later one: against the oracle's iteration stopped by the same test, at the
    capped iterates' 1e-11 (at 1e-10 and below S_L is that iterate to rounding:
    the next change is of the square)."""
    from oracle import rh as R
    b = nk()
    a, be, de = _intervals(n, 3)
    a[-1], be[n - 2], de[n - 2] = 0.05, 0.0, 0.0  # an eigenvalue far from 1: more steps
    T = _dense(a, be, de)
    for scaling, scale in ((b.NK_RH_NONE, None), (b.NK_RH_DET, R.determinant_scale)):
        S, it, _ = R.roberts_higham(T, tol=tol, scale=scale)
        banner(f"tolerance {tol:g} n={n} scaling={scaling}")
        z, info, rc = b.nk_small_sign(n, 0, True, a, be, de, b.nk_sign_params_default(rh_scaling=scaling, rh_tol=tol))
        assert rc == 0 and info.rh_iters == it
        assert np.linalg.norm(z - S[:, 0]) <= 1e-11
        res = np.linalg.norm(S @ S - np.eye(n)) / np.sqrt(n)
        assert abs(info.rh_residual - res) <= 1e-10 + 1e-6 * res


DIMS, MU = (4, 4, 2, 6), 0.3


def _sources(lat, xs, block, **kw):
    b = nk()
    p = b.nk_sign_params_default(mu=MU, nrhs=len(xs), block=block, **kw)
    dx = to_dev(xs)
    dy = torch_cuda().empty_like(dx)
    info, rc = b.nk_sign_apply_device(lat.h, p, dx, dy)
    assert rc == 0
    return to_host(dy).reshape(len(xs), -1), info


def test_loose_tolerance_of_a_batch():
    """Sources of one call that stop at different steps, in lockstep against
    one at a time (k = 60 on this lattice: 1e-9, the tolerance of that
    comparison at k = 100)."""
    lat, _ = make_lattice(DIMS, 0.6, seed=1)
    xs = latgen.random_sources(DIMS, 4, 7)
    for tol in (0.3, 1e-2, 1e-4):
        banner(f"lockstep with tolerance {tol:g}")
        kw = dict(k=60, ell_per_rhs=[2, 9, 20, 30], rh_tol=tol)
        (yb, ib), (ys, i1) = _sources(lat, xs, 1, **kw), _sources(lat, xs, 0, **kw)
        assert ib.rh_iters == i1.rh_iters
        for s in range(len(xs)):
            assert rel(yb[s], ys[s]) < 1e-9, (tol, s)
    lat.close()


@pytest.mark.parametrize("r", [40, 130, 400, 560])
def test_batches_at_the_workspace_bound(r):
    """Plain problems of order 60 by the hundred: nine, eight and six steps in
    closed form, and none, within 512 MB; the others with explicit inverses.
    In lockstep against one at a time (k = 60: 1e-9 as above)."""
    lat, _ = make_lattice(DIMS, 0.6, seed=1)
    xs = latgen.random_sources(DIMS, r, 7)
    banner(f"{r} plain problems in one batch")
    (yb, ib), (ys, i1) = _sources(lat, xs, 1, k=60, ell=0), _sources(lat, xs, 0, k=60, ell=0)
    assert abs(ib.rh_iters - i1.rh_iters) <= 1
    assert max(rel(yb[s], ys[s]) for s in range(r)) < 1e-9
    lat.close()


@pytest.mark.parametrize("n,ell", [(20, 0), (140, 0), (140, 20)])
def test_unnamed_scaling_is_no_scaling(n, ell):
    """nk_small_sign takes any rh_scaling; values that name no scaling iterate
    unscaled (the same steps: the same bits)."""
    b = nk()
    a, be, de = _intervals(n, 5)
    banner(f"unnamed scaling n={n} ell={ell}")
    z0, i0, _ = b.nk_small_sign(n, ell, True, a, be, de, b.nk_sign_params_default())
    for scaling in (-1, 3, 7):
        z, i, rc = b.nk_small_sign(n, ell, True, a, be, de, b.nk_sign_params_default(rh_scaling=scaling))
        assert rc == 0 and i.rh_iters == i0.rh_iters and np.array_equal(z, z0)


@pytest.mark.parametrize("n", [6, 60, 128, 130, 300])
@pytest.mark.parametrize("det", [False, True])
def test_cap_is_reported_only_when_it_ended_the_iteration(n, det):
    """The return code under every cap from 1 to 12, past the steps in closed
    form too: a warning if and only if the stopping test had not held by then,
    with the iterate (1e-11).  The tolerance, 1e-10, lies a factor of 10 or
    more from every change of these iterations."""
    from oracle import rh as R
    b = nk()
    a, be, de = _intervals(n, 3)
    a[-1], be[n - 2], de[n - 2] = 0.05, 0.0, 0.0
    T = _dense(a, be, de)
    scale = R.determinant_scale if det else None
    _, stop, _ = R.roberts_higham(T, tol=1e-10, scale=scale)
    assert 6 < stop < 12
    banner(f"caps n={n} det={det}, stops at {stop}")
    for maxit in range(1, 13):
        S, it, _ = R.roberts_higham(T, tol=1e-10, maxit=maxit, scale=scale)
        p = b.nk_sign_params_default(rh_maxit=maxit, rh_tol=1e-10,
                                     rh_scaling=b.NK_RH_DET if det else b.NK_RH_NONE)
        z, info, rc = b.nk_small_sign(n, 0, True, a, be, de, p)
        assert info.rh_iters == it == min(maxit, stop)
        assert rc == (0 if stop <= maxit else b.NK_WARN_NOTCONV), maxit
        assert np.linalg.norm(z - S[:, 0]) <= 1e-11 * max(1.0, np.linalg.norm(S[:, 0]))


@pytest.mark.parametrize("n", [6, 64, 130, 300])
def test_size_of_the_whole_matrix(n):
    """sgn(f T) e_1 = sgn(T) e_1 with determinant scaling, f down to where the
    products of two entries leave the exponent range and up to where they
    exceed it (condition below 10: 1e-12)."""
    b = nk()
    a, be, de = _intervals(n, 4)
    w, q = np.linalg.eigh(_dense(a, be, de))
    ref = (q * np.sign(w)) @ q[0].conj()
    for f in (1e-200, 1e-165, 1e-156, 1e-120, 1e120, 1e150, 1e165):
        banner(f"matrix times {f:g}, n={n}")
        z, info, rc = b.nk_small_sign(n, 0, True, f * a, f * be, f * de, b.nk_sign_params_default(rh_scaling=b.NK_RH_DET))
        assert rc == 0 and np.linalg.norm(z - ref) < 1e-12, f
