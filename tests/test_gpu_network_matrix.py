"""The FP32 network evaluated by the whole wave on the matrix cores: a trajectory's result may not
depend on its place in the wave, on partly filled waves, on lanes at other phases of mlp_every, or on
the block size asked for (bit for bit), and it follows the FP64 network as FP32 state does elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._gpu import gpu_run  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _ig(n):
    return W.exponential_ig_learned(n_traj=n, seed=51, params=W.mlp_random(17, scale=0.2, out_bias=1.0)).with_(precision=1)


@pytest.mark.parametrize("k", [1, 7, 16])
def test_place_in_the_wave_does_not_matter(k):
    w = _ig(131)
    print(f"network wave place k={k}", flush=True)
    (N, lnw, st), _ = gpu_run(w, mlp_every=k)
    for i in (0, 31, 32, 63, 64, 130):
        (N1, l1, s1), _ = gpu_run(w, n_traj=1, traj_offset=i, mlp_every=k)
        assert N1[0] == N[i] and l1[0] == lnw[i] and s1[0] == st[i], i
    (N64, l64, s64), _ = gpu_run(w.with_(precision=0), mlp_every=k)
    # FP32 state against FP64 on the same streams: the bars of the learned control's coupled test
    same = st == s64
    assert np.mean(np.abs(N - N64) < 1e-4) > 0.98 and same.mean() > 0.95
    assert np.median(np.abs(lnw - l64)[same]) < 1e-5 and np.std(lnw) > 0.05


@pytest.mark.parametrize("k", [3, 7, 64])
def test_refilled_lanes_and_block_sizes(k):
    """20,000 paths on 64-thread blocks are refilled (lanes at other phases than their wave's), on larger
    blocks not; 1024 is above the kernel's own largest block."""
    w = _ig(20_000)
    print(f"network refills k={k}", flush=True)
    a, ha = gpu_run(w, mlp_every=k)
    for block in (64, 1024):
        b, hb = gpu_run(w, mlp_every=k, block_size=block, blocks_per_cu=1)
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
        assert ha["n_steps_total"] == hb["n_steps_total"]
    c, _ = gpu_run(w, mlp_every=k, max_steps=900)      # most paths censored inside a chunk
    early = (a[2] & 0x3fffffff) <= 900
    assert 0 < early.sum() < len(early)
    np.testing.assert_array_equal(a[2][early], c[2][early])
    assert np.all(c[2][~early] == (900 | 0x80000000))
