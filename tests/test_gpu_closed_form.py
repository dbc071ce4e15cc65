"""Roberts-Higham from a tridiagonal matrix in closed form, where it ends and
the iteration with explicit inverses takes over: caps, badly scaled entries,
loose tolerances, wide spectra and the workspace's bound."""
import numpy as np
import pytest

from tests.gpu_helpers import banner, nk

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
