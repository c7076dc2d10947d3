"""The noise-table generators where their split of the work can go wrong, against the oracle's sequential
solves: trajectories whose strides meet the kink at other phases, or may not stride at all, node counts on
both sides of the segment rule and not multiples of a block.  Relative tolerance 1e-9, the tables' parity bar:
both sides take RK4 steps by the same rule, and rounding over 1e5 steps is 1e-11."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402

V0, AP, AM = W.V0, W.A_PLUS, W.A_MINUS


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


# kind, phi_T, A_+, A_-, bump, sigma, n, lo, hi, phi_start, pi_start
MATCHED = {
    # the kink at another phase of the sample grid and of the strides; node counts 65 and 1025 (256 segments)
    "offset_start": (0, 0.0, AP, AM, (0, 0, 0), 0.7, 65, -0.05, 0.01, 1.234567, -0.12),
    "many_nodes": (0, 0.0, AP, 0.3 * AP, (0, 0, 0), 1.0, 1025, -0.3, 0.2, 1.5, -0.12),
    # more nodes than 2^18/128: 64 segments
    "most_nodes": (0, 0.0, AP, AM, (0, 0, 0), 1.0, 4095, -0.05, 0.012, 1.0, -0.12),
    # climbs first, turns and rolls down over the kink
    "turns": (0, 0.0, AP, 0.5 * AP, (0, 0, 0), 1.0, 33, -0.2, 0.02, 0.8, 0.3),
    # starts below the kink, climbs over it, turns and passes it downwards: a kink that no stride may span
    "climbs_over": (0, 0.0, AP, 0.7 * AP, (0, 0, 0), 1.0, 17, -2.0, -1.2, -0.05, 0.6),
    # starts on the kink
    "from_kink": (0, 0.0, AP, 0.9 * AP, (0, 0, 0), 1.0, 17, -1.3, -0.9, 0.0, -0.12),
    # a potential that rises towards smaller phi above the kink: single samples only
    "uphill": (0, 0.0, -0.02 * V0, 0.3 * AP, (0, 0, 0), 1.0, 9, 0.35, 0.4, 1.0, -0.9),
    "exponential": (1, 0.0, 0.3, 0.0, (0, 0, 0), 0.3, 257, 0.0, 1.2, 4.0, -0.3),
    "bump": (2, W.BUMP_PHI0, 0.0, 0.0, W.BUMP, 1.0, 129, W.BUMP_PHI_LO, W.BUMP_PHI_IN, 2.5, -0.03),
}


@pytest.mark.parametrize("name", sorted(MATCHED))
def test_matched_table_equals_sequential_solve(name):
    kind, phi_T, Ap, Am, bump, sigma, n, lo, hi, phi_start, pi_start = MATCHED[name]
    v0 = W.BUMP_V0 if kind == 2 else V0
    print(f"matched {name}", flush=True)
    pot = fpt.make_potential(kind, v0, phi_T, Ap, Am, 3.0, 0.0, 1.0, bump)
    try:
        o = orc.noise_table_matched(kind, v0, phi_T, Ap, Am, sigma, n, lo, hi, phi_start, pi_start, bump=bump)
    except ValueError:
        with pytest.raises(fpt.FptError):
            fpt.fpt_noise_table_matched(pot, sigma, n, lo, hi, phi_start, pi_start)
        return
    g = fpt.fpt_noise_table_matched(pot, sigma, n, lo, hi, phi_start, pi_start)
    np.testing.assert_allclose(g[2], o[2], rtol=1e-9, atol=0)
    np.testing.assert_allclose(g[0], o[0], rtol=1e-9, atol=0)
    np.testing.assert_allclose(g[1], o[1], rtol=0, atol=1e-14)


@pytest.mark.parametrize("t_lo,t_hi,n", [(0.0, 12.5, 2), (-1.5, 3.25, 131), (0.7, 0.7, 1), (0.0, 6.0, 2049)])
def test_time_tables_equal_sequential_solve(t_lo, t_hi, n):
    w = W.srusr_time()
    pot = fpt.make_potential(w.kind, w.V0, w.phi_T, w.A_plus, w.A_minus, w.phi_in, w.pi_in, w.phi_end)
    args = (t_lo, t_hi, *w.match_start, w.phi_in)
    print(f"time nodes {t_lo} {t_hi} {n}", flush=True)
    g = fpt.fpt_noise_table_matched_time(pot, 1.0, n, *args)
    o = orc.noise_table_matched_time(w.kind, w.V0, w.phi_T, w.A_plus, w.A_minus, 1.0, n, *args)
    for k in (0, 2):
        np.testing.assert_allclose(g[k], o[k], rtol=1e-9, atol=0)
    np.testing.assert_allclose(g[3], o[3], rtol=1e-9, atol=1e-12)
    g = fpt.fpt_noise_table_bessel2d_time(pot, 0.1, n, *args)
    o = orc.noise_table_bessel2d_time(w.kind, w.V0, w.phi_T, w.A_plus, w.A_minus, 0.1, n, *args)
    for a, b in zip(g[:3], o[:3]):
        np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * math.sqrt(float(np.mean(np.square(b)))))


@pytest.mark.parametrize("sigma", [1e-3, 0.1, 2.0])
def test_covariance_series_over_sigma(sigma):
    """The series' cut at both ends of its range of sigma, nu from 1.5 (flat) to 2.3 (steep)."""
    print(f"bessel2d sigma {sigma}", flush=True)
    for Ap in (AP, 1.0 * V0):
        pot = fpt.make_potential(0, V0, 0.0, Ap, AM, 0.5, 0.0, -0.01)
        g = fpt.fpt_noise_table_bessel2d(pot, sigma, 67, -0.01, 0.5)
        o = orc.noise_table_bessel2d(0, V0, 0.0, Ap, AM, sigma, 67, -0.01, 0.5)
        for a, b in zip(g, o):
            np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * float(np.max(np.abs(b))) if b is o[1] else 0)
