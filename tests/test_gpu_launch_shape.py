"""A run's default launch shape follows its trajectory count (blocks of one to sixteen waves).  At the
counts where the shape changes, every trajectory equals the run with the block size given, bit for bit,
and the histogram counts every trajectory once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._gpu import gpu_context, gpu_run  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


PROBLEMS = {
    "fp64": lambda: W.linear_slow_roll().with_(dN=2e-2),
    "fp32": lambda: W.exponential_ig(dN=2e-2, A_bias=0.5).with_(precision=1),
    "fp64_2d": lambda: W.exponential_2d(dN=2e-2, A_bias=0.5),
}


@pytest.mark.parametrize("problem", sorted(PROBLEMS))
@pytest.mark.parametrize("waves,extra", [(0, 1), (0, 63), (1, 0), (1, 1), ("cus", -1), ("cus", 1), ("5cus", 7),
                                         ("16cus", -64), ("16cus", 0), ("16cus", 1)])
def test_default_shape_equals_fixed_blocks(problem, waves, extra):
    cus = _cus()
    n = 64 * {"cus": cus, "5cus": 5 * cus, "16cus": 16 * cus}.get(waves, waves) + extra
    w = PROBLEMS[problem]().with_(n_traj=n)
    print(f"launch shape {problem} n={n}", flush=True)
    a, ha = gpu_run(w)
    b, hb = gpu_run(w, block_size=256, blocks_per_cu=2)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)
    assert int(ha["count"].sum()) + ha["n_ended_early"] + ha["n_censored"] == n
    np.testing.assert_array_equal(ha["count"], hb["count"])
    assert ha["n_steps_total"] == hb["n_steps_total"]


def test_shapes_alternate_on_one_context():
    """Runs of different shapes on one context add up: small, large, small."""
    w = W.linear_slow_roll().with_(dN=2e-2)
    ctx = gpu_context(w)
    counts = (65, 64 * 16 * _cus() + 3, 1000)
    off = 0
    for n in counts:
        ctx.run(n, w.dN, w.seed, off)
        off += n
    h = ctx.histogram()
    ctx.destroy()
    _, one = gpu_run(w, n_traj=off, dumps=False)
    np.testing.assert_array_equal(h["count"], one["count"])
    assert h["n_steps_total"] == one["n_steps_total"]
