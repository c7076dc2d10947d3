"""FP32 state on a time table over a potential that falls upwards (equal negative slopes): |V'/V| grows along
the path, so a bound on pi taken between phi_end and phi_T says nothing above phi_T, and the eps_1 = 1 end must
be seen in the step it comes in.  Against the FP64 path on the same streams: the same step on 95 % of the paths
and N there within 1e-4, the bars of the other coupled FP32 tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import fpt  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


# V0, phi_T, phi_in, phi_end with A_+ = A_- = -0.1 (V = 0 at phi = 1): phi_T below the path, between its ends
CASES = {"kink_below": (1.0, -9.0, 0.9, -0.1), "kink_inside": (0.1, 0.0, 0.9, -0.1)}


@pytest.mark.parametrize("dN", [1e-3, 2e-3])
@pytest.mark.parametrize("block", [0, 64])
@pytest.mark.parametrize("name", sorted(CASES))
def test_end_is_seen_in_its_step(name, block, dN):
    V0, phi_T, phi_in, phi_end = CASES[name]
    print(f"fp32 falling {name} block={block} dN={dN}", flush=True)
    n = 2000
    pot = fpt.make_potential(0, V0, phi_T, -0.1, -0.1, phi_in, 0.0, phi_end)
    res = []
    for prec in (fpt.FPT_FP64, fpt.FPT_FP32_STATE):
        ctx = fpt.Context(pot, np.full(5, 0.002), np.full(5, 0.1), 0.0, 10.0, max_steps=20001, precision=prec,
                          axis=fpt.FPT_AXIS_TIME, block_size=block, blocks_per_cu=1 if block else 0)
        out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
        out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
        ctx.run(n, dN, 83, 0, None, *out)
        torch.cuda.synchronize()
        ctx.destroy()
        res.append([out[0].cpu().numpy(), out[2].cpu().numpy().view(np.uint32)])
    (N64, s64), (N32, s32) = res
    assert np.all((s64 & fpt.FPT_FLAG_ENDED_EARLY) != 0)
    same = s64 == s32
    assert same.mean() > 0.95 and np.max(np.abs(N32 - N64)[same]) < 1e-4
