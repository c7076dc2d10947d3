"""Rounding of the 2D noise nodes: the power series summed by recurrence may not be further off than the same
series with every term from its own powers and gamma functions.  The reference is the covariance with 40
digits; the bounds are the root mean square errors of separate terms over these same nodes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mp = pytest.importorskip("mpmath")

from paper_2410_13683_amd import fpt  # noqa: E402

# sigma: rms relative error of Xi_phiphi and of Xi_pipi with separate terms
SEPARATE_TERMS = {0.05: (8.071e-16, 2.032e-13), 0.1: (7.184e-16, 2.666e-14), 1.0: (4.247e-16, 9.042e-16),
                  1.5: (4.932e-16, 7.750e-16), 2.0: (6.698e-16, 1.126e-15)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _exact(sigma, A, phi):
    V = 1 + mp.mpf(A) * mp.mpf(phi)
    nu = mp.sqrt(mp.mpf("2.25") + 3 * (A / V) ** 2)
    s, hs = mp.mpf(sigma), mp.sqrt(mp.pi) / 2
    Ak, Bk = hs * mp.expjpi((nu + 0.5) / 2), hs * mp.expjpi((nu + 1.5) / 2)
    Z = Ak * mp.besselj(nu, s) + Bk * mp.bessely(nu, s)
    dZ = Ak * mp.besselj(nu, s, 1) + Bk * mp.bessely(nu, s, 1)
    F, G = s ** 1.5 * Z, -s * (1.5 * s ** 0.5 * Z + s ** 1.5 * dZ)
    c = V / (6 * mp.pi ** 2)
    return c * abs(F) ** 2, c * abs(G) ** 2


@pytest.mark.parametrize("sigma", sorted(SEPARATE_TERMS))
def test_rounding_is_no_larger_than_of_separate_terms(sigma):
    n, lo, hi = 301, -0.2, 0.5
    h = (hi - lo) / (n - 1)
    print(f"covariance rounding sigma {sigma}", flush=True)
    err = [[], []]
    with mp.workdps(40):
        for A_plus in (0.05, 0.3, 1.0):
            pot = fpt.make_potential(0, 1.0, 0.0, A_plus, 0.3 * A_plus, 0.5, 0.0, lo)
            X = fpt.fpt_noise_table_bessel2d(pot, sigma, n, lo, hi)
            for j in range(0, n, 3):
                phi = lo + j * h
                A = A_plus if phi >= 0 else 0.3 * A_plus
                if abs(np.sqrt(2.25 + 3 * (A / (1 + A * phi)) ** 2) - 2) < 0.05:
                    continue                        # near nu = 2 the form cancels
                for e, x, v in zip(err, (X[0][j], X[2][j]), _exact(sigma, A, phi)):
                    e.append(float((mp.mpf(x) - v) / v))
    assert len(err[0]) == 281
    for e, bound in zip(err, SEPARATE_TERMS[sigma]):
        assert np.sqrt(np.mean(np.square(e))) <= bound
