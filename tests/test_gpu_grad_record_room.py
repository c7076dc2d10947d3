"""Gradient runs whose noise carries the paths over each grid line several times: the records fit in the pool, so
recording takes no longer than sampling and replaying (fpt_mlp_grad_noalloc), and gives the same node weights.
Medians of 5 calls may differ by 15 % (they repeat to 3 %; with too little room recording took 1.3 and 1.4 times
as long)."""
import statistics
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._gpu import gpu_context  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dN,grid_n", [(2e-4, (24, 12)), (2e-3, (64, 16)), (2e-3, (24, 12))])
def test_recording_is_no_slower_than_replay(dN, grid_n, precision):
    n = 250_000
    w = W.exponential_ig_learned(dN=dN, params=W.mlp_random(3), grid_n=grid_n).with_(precision=precision)
    ctx = gpu_context(w)
    res = []
    for noalloc in (False, True):
        g = torch.empty(fpt.FPT_MLP_NPARAM, device="cuda")
        G = torch.empty(grid_n[0] * grid_n[1], dtype=torch.float64, device="cuda")
        ms = []
        for _ in range(7):
            torch.cuda.synchronize()
            t = time.perf_counter()
            J, n_tail = ctx.mlp_grad(n, dN, 3, -10.0, g, d_G=G, noalloc=noalloc)
            ms.append(1e3 * (time.perf_counter() - t))
        res.append((statistics.median(ms[2:]), J, n_tail, G.cpu().numpy()))
    ctx.destroy()
    (t, J, k, G), (t2, J2, k2, G2) = res
    print(f"dN {dN} grid {grid_n} precision {precision}: recorded {t:.2f} ms, replayed {t2:.2f}", flush=True)
    assert k == k2 and k > 0
    # 2.5e5 paths' FP64 sums in another order: 1e-11 of the largest weight is 1e5 roundings
    np.testing.assert_allclose(J, J2, rtol=1e-11)
    np.testing.assert_allclose(G, G2, rtol=0, atol=1e-11 * np.abs(G2).max())
    assert t < 1.15 * t2
