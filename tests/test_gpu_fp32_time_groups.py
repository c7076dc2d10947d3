"""FP32 state on time tables: the plain groups' conditions (below the kink, inside the table, S > 0,
|pi| away from sqrt 2) against the FP64 path on the same streams, on problems whose paths cross each
condition's border mid-run.  The bars are those of the other coupled FP32 tests: N within 1e-4 on 98 %
of the paths, the same step on 95 %, ln w within 1e-5 in the median."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


# A_plus, A_minus, phi_T, phi_in, pi_in, phi_end, t_lo, t_hi, S, tan; V0 = 1, dN = 2e-3
CASES = {
    "noise_ends": (0.3, 0.1, 0.2, 0.1, -0.1, -0.1, 0.0, 0.8, np.r_[np.linspace(0.05, 0.03, 12), 0.0], np.full(13, 0.2)),
    "hole_in_table": (0.3, 0.1, 0.2, 0.1, -0.1, -0.1, 0.0, 2.0, np.array([0.05, 0.04, 0.0, 0.0, 0.05, 0.04]), np.full(6, 0.2)),
    "starts_late": (0.3, 0.1, 0.2, 0.1, -0.1, -0.1, 0.3, 2.0, np.linspace(0.05, 0.03, 9), np.linspace(0.3, -0.2, 9)),
    "before_zero": (0.3, 0.1, 0.2, 0.1, -0.1, -0.1, -0.5, 0.7, np.linspace(0.05, 0.03, 9), np.full(9, 0.1)),
    "hops_over_kink": (0.5, 0.1, 0.1, 0.12, 0.0, -0.15, 0.0, 5.0, np.linspace(0.06, 0.04, 33), np.full(33, 0.3)),
    # paths end at eps_1 = 1 or cross, through the table's pi noise
    "near_end": (1.3, 1.3, 0.5, 1.0, -1.1, 0.0, 0.0, 2.0, np.full(5, 0.1), np.full(5, -1.5)),
}


@pytest.mark.parametrize("A", [0.0, 0.7])
@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("block", [0, 64])
def test_plain_time_groups_follow_fp64(name, A, block):
    Ap, Am, phi_T, phi_in, pi_in, phi_end, lo, hi, S, t = CASES[name]
    print(f"fp32 time groups {name} A={A} block={block}", flush=True)
    n, dN, seed = 4000, 2e-3, 79
    pot = fpt.make_potential(0, 1.0, phi_T, Ap, Am, phi_in, pi_in, phi_end)
    res = []
    for prec in (fpt.FPT_FP64, fpt.FPT_FP32_STATE):
        ctx = fpt.Context(pot, S, t, lo, hi, bias_kind=W.BIAS_CONST if A else W.BIAS_NONE, A=A, max_steps=20001,
                          precision=prec, axis=fpt.FPT_AXIS_TIME, block_size=block, blocks_per_cu=1 if block else 0)
        out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
        out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
        ctx.run(n, dN, seed, 0, None, *out)
        torch.cuda.synchronize()
        ctx.destroy()
        res.append([out[0].cpu().numpy(), out[1].cpu().numpy(), out[2].cpu().numpy().view(np.uint32)])
    (N64, l64, s64), (N32, l32, s32) = res
    same = s64 == s32
    assert same.mean() > 0.95 and np.mean(np.abs(N32 - N64)[same & np.isfinite(N64)] < 1e-4) > 0.98
    assert np.median(np.abs(l32 - l64)[same]) < 1e-5
    if name == "near_end":
        early = (s64 & fpt.FPT_FLAG_ENDED_EARLY) != 0
        assert 0.05 < early.mean() < 0.999
