"""The batch's general launch as a captured graph, replayed with other seeds, offsets, counts, steps and work
lists, alone and in turn with small batches on paired waves, which share its item buffers: after every run each
instance's histogram equals the one of single runs over the same trajectories (counts and step totals exactly,
FP64 sums up to the order of the atomic adds: rtol 1e-11)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import runner  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _instances(precision):
    """Some 380 steps at dN = 2e-2; a step cap, a bias and narrow bins among them."""
    ws = [W.linear_slow_roll(),
          W.exponential_ig().with_(bias_kind=W.BIAS_CONST, A_bias=0.5, extra={"instance": 3}),
          W.linear_slow_roll().with_(max_steps=200, n_bins=8, extra={"instance": 9})]
    return [w.with_(precision=precision) for w in ws]


def _play(ws, plan, **options):
    """Run the plan on one batch; after each run compare with single runs on contexts of their own."""
    stream = torch.cuda.Stream()
    ctxs = [runner.context_for(w) for w in ws]
    ref = [runner.context_for(w) for w in ws]
    b = fpt.Batch(ctxs, use_graph=True, **options)
    for k, (seed, off, dN, counts) in enumerate(plan):
        print(f"run {k}: seed {seed} offset {off} dN {dN} counts {counts} {options}", flush=True)
        b.run(counts, dN, seed, off, stream)
        stream.synchronize()
        for c, n in zip(ref, counts):
            c.run(n, dN, seed, off, torch.cuda.current_stream())
        torch.cuda.synchronize()
        for c, r in zip(ctxs, ref):
            h, s = c.histogram(), r.histogram()
            for key in ("n_traj", "n_censored", "n_ended_early", "n_steps_total"):
                assert h[key] == s[key], (k, key)
            np.testing.assert_array_equal(h["count"], s["count"])
            for key in ("sum_w", "sum_w2", "sum_lnw", "sum_lnw2"):
                np.testing.assert_allclose(h[key], s[key], rtol=1e-11, atol=1e-300)
        if k == 1:
            torch.zeros(1 << 20, device="cuda").add_(1.0)      # eager work between two replays
    b.destroy()
    for c in ctxs + ref:
        c.destroy()


@pytest.mark.parametrize("precision", [0, 1])
def test_graph_replays_with_other_work(precision):
    """A given block size keeps the general launch, so every run after the first replays the graph, until a
    longer work list needs a larger buffer and a new capture."""
    plan = [(5, 0, 2e-2, [900, 400, 300]), (6, 10_000, 2e-2, [1200, 50, 0]), (7, 20_000, 1e-2, [64, 640, 333]),
            (8, 0, 2e-2, [0, 0, 1]), (9, 1 << 33, 2e-2, [20_000, 9000, 7000]), (5, 1 << 33, 2e-2, [1, 2, 3])]
    _play(_instances(precision), plan, block_size=256, item_size=256)


@pytest.mark.parametrize("precision", [0, 1])
def test_graph_in_turn_with_paired_launches(precision):
    """Counts on both sides of the paired launch's limit, 512 trajectories per compute unit."""
    over = 512 * torch.cuda.get_device_properties(0).multi_processor_count + 64
    plan = [(5, 0, 2e-2, [over, 400, 300]), (6, 10_000, 2e-2, [500, 50, 0]), (7, 20_000, 2e-2, [300, over, 0]),
            (8, 0, 1e-2, [100, 0, 100]), (9, 5, 2e-2, [over, over, over]), (9, 5, 2e-2, [64, 65, 1])]
    _play(_instances(precision), plan)


def test_tuned_configuration_runs(tmp_path):
    """The tuned block size and chunk on counts that take them, by the graph, twice."""
    over = 512 * torch.cuda.get_device_properties(0).multi_processor_count + 64
    ws = _instances(1)
    stream = torch.cuda.Stream()
    ctxs = [runner.context_for(w) for w in ws]
    ref = [runner.context_for(w) for w in ws]
    b = fpt.Batch(ctxs, use_graph=True)
    counts = [over, 1000, 20_000]
    b.autotune(counts, 2e-2, 3, str(tmp_path / "tune.txt"), torch.cuda.current_stream())
    print(f"tuned {b.config()}", flush=True)
    for seed in (3, 4):
        b.run(counts, 2e-2, seed, 0, stream)
        stream.synchronize()
        for c, r, n in zip(ctxs, ref, counts):
            r.run(n, 2e-2, seed, 0, torch.cuda.current_stream())
            torch.cuda.synchronize()
            h, s = c.histogram(), r.histogram()
            np.testing.assert_array_equal(h["count"], s["count"])
            assert h["n_steps_total"] == s["n_steps_total"] and h["n_traj"] == s["n_traj"]
    b.destroy()
    for c in ctxs + ref:
        c.destroy()
