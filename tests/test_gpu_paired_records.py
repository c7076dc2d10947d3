"""The recording gradient run on paired waves against the same run on fixed (unpaired) blocks: the same
paths, so the tail's count exactly and the node weights to the order of their FP64 sums, at the counts
where the pairs per block change."""
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


CASES = {
    "table_noise": lambda: W.srusr_learned(n_traj=1, A_init=1.8).with_(
        dN=2e-3, mlp_params=W.mlp_random(22, scale=0.1, out_bias=1.8)),
    "constant_noise": lambda: W.exponential_ig_learned(seed=61, dN=2e-3, grid_n=(24, 12),
                                                       params=W.mlp_random(21, scale=0.2, out_bias=1.0)),
}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", sorted(CASES))
def test_paired_records_equal_unpaired(name, precision):
    w = CASES[name]().with_(precision=precision)
    full = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    a, b = gpu_context(w), gpu_context(w, block_size=256, blocks_per_cu=2)
    for n in (1, 64, full + 1, 4 * full + 1, 8 * full, 8 * full + 1):
        print(f"paired records {name} precision={precision} n={n}", flush=True)
        out = []
        for ctx in (a, b):
            g = torch.full((fpt.FPT_MLP_NPARAM,), -1.0, device="cuda")
            G = torch.full((w.grid_n[0] * w.grid_n[1],), -1.0, dtype=torch.float64, device="cuda")
            J, n_tail = ctx.mlp_grad(n, w.dN, w.seed, -10.0, g, traj_offset=(1 << 33) + 3, d_G=G)
            out.append((J, n_tail, G.cpu().numpy()))
        (J, k, G), (J2, k2, G2) = out
        assert k == k2 and k > 0
        # up to 1.3e5 paths' FP64 sums in another order: 1e-11 of the largest weight is 1e5 roundings
        np.testing.assert_allclose(J, J2, rtol=1e-11)
        np.testing.assert_allclose(G, G2, rtol=0, atol=1e-11 * np.abs(G2).max())
    a.destroy()
    b.destroy()
