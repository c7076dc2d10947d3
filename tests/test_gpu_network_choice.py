"""The FP32 network on either of its kernels (matrix cores up to two waves per SIMD and where a wave evaluates
often, scalar weights beyond): a large run equals the same trajectories run in parts small enough for the
matrix cores, bit for bit, and a network that is hardly ever evaluated costs little more than its table."""
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


def _two_waves():
    return 512 * torch.cuda.get_device_properties(0).multi_processor_count


# interval, chunk, count in units of two waves per SIMD, steps per e-fold
@pytest.mark.parametrize("k,chunk,size,dN", [(24, 0, 1.5, 2e-2), (24, 0, 2.5, 2e-2), (128, 0, 1.0, 1e-2), (128, 0, 1.01, 1e-2),
                                             (128, 0, 3.0, 1e-2), (64, 0, 3.0, 1e-2), (64, 0, 6.01, 2e-2), (64, 32, 2.5, 2e-2),
                                             (5, 64, 1.5, 2e-2)])
def test_large_run_equals_its_parts(k, chunk, size, dN):
    n, part = int(size * _two_waves()) + 3, _two_waves()
    w = W.exponential_ig_learned(n_traj=n, dN=dN, params=W.mlp_random(17, scale=0.2, out_bias=1.0)).with_(precision=1)
    print(f"network k={k} chunk={chunk} n={n}", flush=True)
    whole, hist = gpu_run(w, mlp_every=k, chunk=chunk)
    steps = 0
    for off in range(0, n, part):
        m = min(part, n - off)
        out, h = gpu_run(w, n_traj=m, traj_offset=off, mlp_every=k, chunk=chunk)
        for a, b in zip(whole, out):
            np.testing.assert_array_equal(a[off:off + m], b)
        steps += h["n_steps_total"]
    assert hist["n_steps_total"] == steps
    assert np.std(whole[1]) > 0.05


def test_rare_evaluations_cost_little():
    """Every 1024 steps: 1.2 to 1.5 times the tabulated control's time on scalar weights; on the matrix cores, whose two
    waves per SIMD the steps in between do not need, 1.9 to 2.2 times."""
    n = 3 * _two_waves()
    w = W.srusr_learned()
    ms = []
    for every in (0, 1024):
        ctx = gpu_context(w, mlp_every=every)
        t = []
        for r in range(4):
            ctx.run(n, 4 * w.dN, 5 + r, 0, None)
            t.append(ctx.last_kernel_ms())
        ctx.destroy()
        ms.append(min(t[1:]))
    print(f"tabulated {ms[0]:.2f} ms, network every 1024 steps {ms[1]:.2f} ms", flush=True)
    assert ms[1] < 1.7 * ms[0]
