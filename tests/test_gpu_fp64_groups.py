"""The FP64 step groups' variants against the oracle, per trajectory: groups without noise that a path
leaves again (it climbs into the noise window from below), groups on one side of the kink while paths
hop over it, and table lookups on, beside and beyond the table.  Tolerances: the FP64 parity rules."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._glue import assert_fp64_parity  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _ramp(n, lo, hi):
    return np.linspace(lo, hi, n)


# A_plus, A_minus, phi_T, phi_in, pi_in, phi_end, table lo, hi, S, tan; V0 = 1, dN = 2e-3
CASES = {
    # below the window with S = 0, climbs into it and rolls back out
    "climbs_into_window": (0.3, 0.3, -9.0, -0.05, 0.4, -0.5, 0.0, 1.0, np.r_[0.0, _ramp(16, 0.02, 0.05)], _ramp(17, 0.1, 0.3)),
    # noise-free start right under the window's edge, moving along it
    "skims_edge": (0.05, 0.05, -9.0, -1e-4, 0.02, -0.1, 0.0, 0.5, np.r_[0.0, _ramp(4, 0.03, 0.03)], np.zeros(5)),
    # paths hop over the kink, which sits between two nodes
    "hops_over_kink": (0.5, 0.1, 0.1, 0.15, 0.0, -0.15, -0.2, 0.3, _ramp(9, 0.04, 0.06), _ramp(9, 0.3, -0.2)),
    "kink_on_node": (0.5, 0.1, 0.05, 0.06, -0.1, -0.15, -0.2, 0.3, _ramp(11, 0.03, 0.06), np.full(11, 0.2)),
    # both ends of the table inside the paths' range; two nodes only
    "beyond_both_ends": (0.2, 0.2, -9.0, 0.4, -0.1, -0.4, -0.05, 0.05, np.array([0.05, 0.02]), np.array([0.1, 0.4])),
    # no noise anywhere
    "all_quiet": (0.2, 0.1, 0.0, 0.3, -0.1, -0.2, -0.5, -0.4, np.array([0.0, 0.0]), np.array([0.1, 0.4])),
}


@pytest.mark.parametrize("A", [0.0, 0.7])
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("block", [0, 64])
def test_fp64_group_variants(name, A, block):
    Ap, Am, phi_T, phi_in, pi_in, phi_end, lo, hi, S, t = CASES[name]
    print(f"fp64 groups {name} A={A} block={block}", flush=True)
    n, dN, seed = 1000, 2e-3, 77
    w = W.linear_slow_roll().with_(phi_in=phi_in, pi_in=pi_in, phi_end=phi_end, dN=dN, n_traj=n)
    bias = W.BIAS_CONST if A else W.BIAS_NONE
    pot = fpt.make_potential(0, 1.0, phi_T, Ap, Am, phi_in, pi_in, phi_end)
    ctx = fpt.Context(pot, S, t, lo, hi, bias_kind=bias, A=A, max_steps=20000, block_size=block,
                      blocks_per_cu=1 if block else 0)
    out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
    ctx.run(n, dN, seed, 0, None, *out)
    torch.cuda.synchronize()
    ctx.destroy()
    N, lnw, st = (x.cpu().numpy() for x in out)
    p = orc.Problem(kind=0, V0=1.0, phi_T=phi_T, A_plus=Ap, A_minus=Am, phi_in=phi_in, pi_in=pi_in, phi_end=phi_end,
                    S=S, tan_theta=t, phi_lo=lo, phi_hi=hi, bias_kind=bias, A_bias=A)
    ora = orc.run(p, dN, seed, n, max_steps=20000, last_phi=True)
    assert np.mean((ora[2] & orc.FLAG_CENSORED) != 0) < 0.9
    assert_fp64_parity((N, lnw, st.view(np.uint32)), ora, w)


@pytest.mark.parametrize("A", [0.0, 0.7])
@pytest.mark.parametrize("name", ["hops_over_kink", "beyond_both_ends"])
def test_fp64_2d_group_variants(name, A):
    Ap, Am, phi_T, phi_in, pi_in, phi_end, lo, hi, S, t = CASES[name]
    print(f"fp64 2d groups {name} A={A}", flush=True)
    n, dN, seed = 1000, 2e-3, 78
    w = W.linear_slow_roll().with_(phi_in=phi_in, pi_in=pi_in, phi_end=phi_end, dN=dN, n_traj=n)
    X = (S * S, 0.3 * S * S, 0.5 * S * S)
    bias = W.BIAS_CONST if A else W.BIAS_NONE
    pot = fpt.make_potential(0, 1.0, phi_T, Ap, Am, phi_in, pi_in, phi_end)
    ctx = fpt.Context(pot, None, None, lo, hi, Xi=X, bias_kind=bias, A=A, max_steps=20000)
    out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
    ctx.run(n, dN, seed, 0, None, *out)
    torch.cuda.synchronize()
    ctx.destroy()
    N, lnw, st = (x.cpu().numpy() for x in out)
    p = orc.Problem2D(kind=0, V0=1.0, phi_T=phi_T, A_plus=Ap, A_minus=Am, phi_in=phi_in, pi_in=pi_in, phi_end=phi_end,
                      Xpp=X[0], Xpq=X[1], Xqq=X[2], phi_lo=lo, phi_hi=hi, bias_kind=bias, A_bias=A)
    ora = orc.run2d(p, dN, seed, n, max_steps=20000, last_phi=True)
    assert np.mean((ora[2] & orc.FLAG_CENSORED) != 0) < 0.9
    assert_fp64_parity((N, lnw, st.view(np.uint32)), ora, w)
