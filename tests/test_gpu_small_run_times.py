"""Small runs by the default launch, on paired waves or not, take no longer than on the caller's own blocks of
1024 threads: every precision, noise dimension and axis, with and without a bias, on broad paths of some 1600
and 2900 steps.  The medians of 7 kernel times may differ by 20 % (they repeat to 3 %; the fault that this
found was a factor of 1.5 to 1.8)."""
import statistics

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


def _median_ms(n, dim, axis, precision, A, **shape):
    S = np.full(65, 0.05)
    pot = fpt.make_potential(0, 1.0, -9.0, 0.05, 0.05, 0.1, -0.05, 0.0)
    lo, hi = (-0.5, 0.7) if axis == fpt.FPT_AXIS_PHI else (0.0, 40.0)
    noise = dict(Xi=(S * S, 0.3 * S * S, 0.5 * S * S)) if dim == 2 else {}
    ctx = fpt.Context(pot, S, np.full(65, 0.1), lo, hi, bias_kind=fpt.FPT_BIAS_CONST if A else fpt.FPT_BIAS_NONE, A=A,
                      precision=precision, max_steps=1 << 16, lo=-4.0, hi=16.0, axis=axis, **noise, **shape)
    ms = []
    for k in range(9):
        ctx.run(n, 1e-3, 5 + k, 0, None)
        ms.append(ctx.last_kernel_ms())
    ctx.destroy()
    return statistics.median(ms[2:])


@pytest.mark.parametrize("A", [0.0, -0.5])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("dim", [1, 2])
def test_default_launch_is_no_slower_than_full_blocks(dim, axis, precision, A):
    for n in (1000, 32768):
        default = _median_ms(n, dim, axis, precision, A)
        blocks = _median_ms(n, dim, axis, precision, A, block_size=1024)
        print(f"dim {dim} axis {axis} precision {precision} A {A} n {n}: {default:.3f} ms, blocks {blocks:.3f}", flush=True)
        assert default < 1.2 * blocks
