"""Paired waves (a small run's integrating waves take their normals from partner waves): per trajectory
and in the histogram the same as the unpaired kernel on fixed blocks, bit for bit, on every table kind,
bias and potential, at the counts where the pairs per block change, with step caps inside a turn."""
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


def _is(w, A):
    return w.with_(bias_kind=W.BIAS_CONST if A else W.BIAS_NONE, A_bias=A)


PROBLEMS = {
    "fp64_phi": lambda: _is(W.srusr_bessel(), 0.0),
    "fp64_phi_bias": lambda: _is(W.srusr_bessel(), 1.0),
    "fp32_phi": lambda: _is(W.srusr_bessel(), 0.0).with_(precision=1),
    "fp32_phi_bias": lambda: W.srusr_is_fp32(A_bias=2.0),
    "fp64_time": lambda: _is(W.srusr_time(tau_hi=6.0), 0.0),           # noise that stops: nodes with S = 0
    "fp64_time_bias": lambda: _is(W.srusr_time(tau_hi=6.0), 1.0),
    "fp32_time": lambda: _is(W.srusr_time(tau_hi=6.0), 0.0).with_(precision=1),
    "fp32_time_bias": lambda: W.srusr_is_fp32_time(),
    "bump": lambda: W.gaussian_bump(),
    "bump_bias": lambda: W.gaussian_bump_is(),
    "bump_time": lambda: W.gaussian_bump_time(A_bias=3.0),
    "fp64_const": lambda: W.exponential_ig(A_bias=0.5),
    "fp32_const": lambda: W.exponential_ig().with_(precision=1),
    # a steep exponential: epsilon_1 = 1 before phi_end on most paths
    "fp64_early": lambda: W.exponential_ig(alpha=1.3, S=0.05, A_bias=0.2).with_(pi_in=-1.2),
    "fp32_early": lambda: W.exponential_ig(alpha=1.3, S=0.05).with_(pi_in=-1.2, precision=1),
}


def _run(ctx, w, n, off):
    out = [torch.full((n,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
    out.append(torch.zeros(n, dtype=torch.int32, device="cuda"))
    ctx.run(n, w.dN, w.seed, off, torch.cuda.current_stream(), *out)
    h = ctx.histogram()
    return [x.cpu().numpy() for x in out], h


@pytest.mark.parametrize("problem", sorted(PROBLEMS))
def test_paired_equals_unpaired(problem):
    w = PROBLEMS[problem]()
    w = w.with_(dN=w.dN * 20)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    full = 64 * cus
    a, b = gpu_context(w), gpu_context(w, block_size=256, blocks_per_cu=2)
    # 1 to 8 pairs per block, the odd counts above 4, and the first count without pairs
    for n in (1, 64, 65, full, full + 1, 3 * full, 4 * full + 1, 6 * full + 7, 8 * full, 8 * full + 1):
        print(f"paired {problem} n={n}", flush=True)
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
    a.destroy()
    b.destroy()


@pytest.mark.parametrize("problem", ["fp64_phi", "fp32_phi_bias", "fp32_time", "fp64_const", "fp64_early"])
@pytest.mark.parametrize("cap", [1, 7, 8, 16, 17, 333])
def test_step_cap_inside_a_turn(problem, cap):
    w = PROBLEMS[problem]()
    w = w.with_(dN=w.dN * 20, max_steps=cap)
    print(f"paired cap {problem} {cap}", flush=True)
    a, b = gpu_context(w), gpu_context(w, block_size=64, blocks_per_cu=1)
    (x, hx), (y, hy) = _run(a, w, 130, 0), _run(b, w, 130, 0)
    a.destroy()
    b.destroy()
    for u, v in zip(x, y):
        np.testing.assert_array_equal(u, v)
    assert hx["n_censored"] == hy["n_censored"] and (cap > 100 or hx["n_censored"] > 0)


def _batch_counts(pairs, cus):
    """Counts that just fit `pairs` pairs per block on one block per CU, ragged slices among them."""
    lanes = 64 * pairs
    counts = [1, 0, lanes - 1, lanes, lanes + 1, 63]
    used = sum(-(-n // lanes) for n in counts)
    return counts + [(cus - used) * lanes - 5]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("pairs", [1, 2, 3, 4, 6, 8, 9])
def test_small_batch_equals_single_runs(precision, pairs):
    """Batches at the counts where the pairs per block change, and one past the last (9: the general
    kernel): per instance the counts, flags and step total of its own run."""
    from paper_2410_13683_amd import fpt
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    counts = _batch_counts(pairs, cus)
    ws = [_is(W.srusr_bessel(), (0.0, 1.0)[i % 2]).with_(precision=precision, phi_end=-0.01 - 0.004 * i,
                                                          dN=2e-3, max_steps=2500, extra={"instance": i})
          for i in range(len(counts))]
    print(f"small batch precision={precision} pairs={pairs} total={sum(counts)}", flush=True)
    ctxs = [gpu_context(w) for w in ws]
    stream = torch.cuda.Stream()
    batch = fpt.Batch(ctxs, use_graph=True)
    off = (1 << 32) - 100
    for _ in range(2):                       # twice: new work lists on the same batch
        for c in ctxs:
            c.reset()
        batch.run(np.array(counts, dtype=np.uint64), ws[0].dN, ws[0].seed, off, stream=stream)
        hb = [c.histogram() for c in ctxs]
    for i, (w, n) in enumerate(zip(ws, counts)):
        one = gpu_context(w, block_size=256, blocks_per_cu=2)
        if n:
            one.run(n, w.dN, w.seed, off)
        h = one.histogram()
        one.destroy()
        np.testing.assert_array_equal(hb[i]["count"], h["count"])
        for k in ("n_traj", "n_censored", "n_ended_early", "n_steps_total"):
            assert hb[i][k] == h[k], (i, k)
        np.testing.assert_allclose(hb[i]["sum_lnw2"], h["sum_lnw2"], rtol=1e-12, atol=0)
    batch.destroy()
    for c in ctxs:
        c.destroy()
