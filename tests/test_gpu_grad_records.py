"""The gradient from recorded sums (fpt_mlp_grad) against the replayed one (fpt_mlp_grad_noalloc) on the
same paths: the node weights agree to the order of their FP64 sums, the tail's count exactly.  The paths
make no, some or (nearly) all more records than the pool has room for, or are not in the tail at all."""
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


def _ig(dN, grid_n=(24, 12)):
    return W.exponential_ig_learned(seed=61, dN=dN, params=W.mlp_random(21, scale=0.2, out_bias=1.0), grid_n=grid_n)


def _srusr():
    return W.srusr_learned(n_traj=1, A_init=1.8).with_(dN=2e-3, mlp_params=W.mlp_random(22, scale=0.1, out_bias=1.8))


CASES = {
    "few_records": (lambda: _ig(1e-2, (8, 4)), -10.0),
    "most_overflow": (lambda: _ig(1e-4, (64, 4)), -10.0),       # noise hops over every grid line many times
    "some_overflow": (lambda: _ig(2e-3, (40, 4)), -10.0),
    "table_noise": (_srusr, -10.0),
    "table_noise_empty_tail": (_srusr, 0.03),                   # the coarse step's N lie below it
    "empty_tail": (lambda: _ig(2e-3), 1e3),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [1, 65, 3000])
@pytest.mark.parametrize("name", sorted(CASES))
def test_recorded_gradient_equals_replay(name, n, precision):
    make, tail_lo = CASES[name]
    w = make().with_(precision=precision)
    print(f"grad records {name} n={n} precision={precision}", flush=True)
    ctx = gpu_context(w)
    out = []
    for noalloc in (False, True):
        g = torch.full((fpt.FPT_MLP_NPARAM,), -1.0, device="cuda")
        G = torch.full((w.grid_n[0] * w.grid_n[1],), -1.0, dtype=torch.float64, device="cuda")
        J, n_tail = ctx.mlp_grad(n, w.dN, w.seed, tail_lo, g, traj_offset=(1 << 33) + 3, d_G=G, noalloc=noalloc)
        out.append((J, n_tail, g.cpu().numpy(), G.cpu().numpy()))
    ctx.destroy()
    (J, k, g, G), (J2, k2, g2, G2) = out
    assert k == k2 and (k > 0) == (not name.endswith("empty_tail") and (n > 1 or k2 > 0))
    # sums of at most 3000 x 1e5 terms in another order: 1e-12 of the largest weight leaves room for their
    # rounding (a random walk of 1e-16 each)
    np.testing.assert_allclose(J, J2, rtol=1e-12)
    np.testing.assert_allclose(G, G2, rtol=0, atol=1e-12 * max(np.abs(G2).max(), 1e-300))
    np.testing.assert_allclose(g, g2, rtol=0, atol=3e-7 * max(np.abs(g2).max(), 1e-30))
