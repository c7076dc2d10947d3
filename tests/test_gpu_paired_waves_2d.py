"""Paired waves with 2D noise: per trajectory and in the histogram the same as the unpaired kernel on
fixed blocks, bit for bit, in both precisions, with and without bias, on both axes, at the counts where
the pairs per block change and with step caps inside a turn."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._gpu import gpu_context  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _run(ctx, w, n, off):
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
    out.append(torch.zeros(n, dtype=torch.int32, device="cuda"))
    ctx.run(n, w.dN, w.seed, off, torch.cuda.current_stream(), *out)
    h = ctx.histogram()
    return [x.cpu().numpy() for x in out], h


def _same(a, b, w, n):
    a.reset()
    b.reset()
    (x, hx), (y, hy) = _run(a, w, n, (1 << 33) + 5), _run(b, w, n, (1 << 33) + 5)
    for u, v in zip(x, y):
        np.testing.assert_array_equal(u, v)
    np.testing.assert_array_equal(hx["count"], hy["count"])
    for k in ("n_traj", "n_censored", "n_ended_early", "n_steps_total"):
        assert hx[k] == hy[k], k
    for k in ("sum_w", "sum_lnw2"):
        np.testing.assert_allclose(hx[k], hy[k], rtol=1e-12, atol=0)
    return hx


def _problem(precision, A, axis):
    w = W.srusr_2d() if axis == "phi" else W.srusr_2d_time()
    return w.with_(precision=precision, bias_kind=W.BIAS_CONST if A else W.BIAS_NONE, A_bias=A, dN=w.dN * 20)


@pytest.mark.parametrize("axis", ["phi", "time"])
@pytest.mark.parametrize("A", [0.0, 1.0])
@pytest.mark.parametrize("precision", [0, 1])
def test_paired_equals_unpaired_2d(precision, A, axis):
    w = _problem(precision, A, axis)
    full = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    a, b = gpu_context(w), gpu_context(w, block_size=256, blocks_per_cu=2)
    # 1 to 8 pairs per block, an odd count above 4, and the first count without pairs
    for n in (1, 65, full + 1, 4 * full + 1, 8 * full, 8 * full + 1):
        print(f"paired 2d precision={precision} A={A} {axis} n={n}", flush=True)
        _same(a, b, w, n)
    a.destroy()
    b.destroy()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cap", [1, 3, 8, 9, 16, 333])
def test_step_cap_inside_a_turn_2d(precision, cap):
    w = _problem(precision, 0.0, "phi").with_(max_steps=cap)
    print(f"paired 2d cap precision={precision} cap={cap}", flush=True)
    a, b = gpu_context(w), gpu_context(w, block_size=64, blocks_per_cu=1)
    h = _same(a, b, w, 200)
    assert cap > 100 or h["n_censored"] > 0
    a.destroy()
    b.destroy()
