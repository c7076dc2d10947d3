"""Cases that enter the routes they are for: matched nodes behind a rising potential (single-sample strides), FP64
groups without noise for a whole path, and every width of an unpaired block."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2410_13683_amd import fpt  # noqa: E402
from paper_2410_13683_amd import workloads as W  # noqa: E402
from tests._glue import assert_fp64_parity  # noqa: E402
from tests._gpu import gpu_run  # noqa: E402

V0 = W.V0


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("A_plus", [-1e-9 * V0, -0.02 * V0])
def test_matched_nodes_after_a_rising_potential(A_plus):
    """A_+ < 0: the trajectory is thrown over phi_T and rolls down the lower branch, where its nodes are; all of
    them are matched.  Tolerance: the tables' parity bar."""
    print(f"matched after A_+ = {A_plus}", flush=True)
    A_minus, lo, hi, start = 0.3 * W.A_PLUS, -0.9, -0.8, (0.05, -0.9)
    pot = fpt.make_potential(0, V0, 0.0, A_plus, A_minus, 3.0, 0.0, 1.0)
    o = orc.noise_table_matched(0, V0, 0.0, A_plus, A_minus, 1.0, 33, lo, hi, *start)
    g = fpt.fpt_noise_table_matched(pot, 1.0, 33, lo, hi, *start)
    assert np.all(o[2] != 1.0)
    for a, b in zip(g, o):
        np.testing.assert_allclose(a, b, rtol=1e-9, atol=0)


# table lo, hi, S: no noise, the whole path below the table; the same, noise at the nodes above the lowest
QUIET = {"no_noise": (0.5, 0.6, [0.0, 0.0]), "noise_above": (0.35, 0.6, [0.0, 0.05, 0.05]),
         "enters_from_noise": (0.2, 0.6, [0.0, 0.05, 0.05])}


@pytest.mark.parametrize("A", [0.0, 0.7])
@pytest.mark.parametrize("name", sorted(QUIET))
@pytest.mark.parametrize("block", [0, 64])
def test_paths_without_noise(name, A, block):
    """Paths from phi = 0.3 to -0.2, below a phi table that ends on S = 0, or into that region."""
    lo, hi, S = QUIET[name]
    S, t = np.array(S), np.full(len(S), 0.2)
    print(f"quiet {name} A={A} block={block}", flush=True)
    n, dN, phi_in, pi_in, phi_end = 300, 2e-3, 0.3, -0.1, -0.2
    pot = fpt.make_potential(0, 1.0, 0.0, 0.2, 0.1, phi_in, pi_in, phi_end)
    bias = W.BIAS_CONST if A else W.BIAS_NONE
    ctx = fpt.Context(pot, S, t, lo, hi, bias_kind=bias, A=A, max_steps=20000, block_size=block,
                      blocks_per_cu=1 if block else 0)
    out = [torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2)]
    out.append(torch.empty(n, dtype=torch.int32, device="cuda"))
    ctx.run(n, dN, 7, 0, None, *out)
    torch.cuda.synchronize()
    ctx.destroy()
    N, lnw, st = (x.cpu().numpy() for x in out)
    p = orc.Problem(kind=0, V0=1.0, phi_T=0.0, A_plus=0.2, A_minus=0.1, phi_in=phi_in, pi_in=pi_in, phi_end=phi_end,
                    S=S, tan_theta=t, phi_lo=lo, phi_hi=hi, bias_kind=bias, A_bias=A)
    ora = orc.run(p, dN, 7, n, max_steps=20000, last_phi=True)
    assert (len(np.unique(ora[2])) == 1) == (name != "enters_from_noise")
    w = W.linear_slow_roll().with_(phi_in=phi_in, pi_in=pi_in, phi_end=phi_end, dN=dN, n_traj=n)
    assert_fp64_parity((N, lnw, st.view(np.uint32)), ora, w)


# problems without a paired kernel, whose default shape follows the count from one wave on; and those with one,
# above its largest count
UNPAIRED = {
    "tabulated_fp64": (0, lambda: W.exponential_ig_learned(dN=2e-2, params=W.mlp_random(3)), {}),
    "tabulated_fp32": (0, lambda: W.exponential_ig_learned(dN=2e-2, params=W.mlp_random(3)).with_(precision=1), {}),
    "network_fp64": (0, lambda: W.exponential_ig_learned(dN=5e-2, params=W.mlp_random(3)), {"mlp_every": 16}),
    "network_fp32": (0, lambda: W.exponential_ig_learned(dN=2e-2, params=W.mlp_random(3)).with_(precision=1), {"mlp_every": 16}),
    "time_2d_fp32": (0, lambda: W.srusr_2d_time().with_(precision=1, max_steps=400), {}),
    "fp64": (8, lambda: W.linear_slow_roll().with_(dN=2e-2), {}),
    "fp32": (8, lambda: W.exponential_ig(dN=2e-2, A_bias=0.5).with_(precision=1), {}),
    "fp64_2d": (8, lambda: W.exponential_2d(dN=2e-2, A_bias=0.5), {}),
    "fp32_2d": (8, lambda: W.exponential_2d(dN=2e-2, A_bias=0.5).with_(precision=1), {}),
}


@pytest.mark.parametrize("name,waves_per_cu", [(name, k) for name in sorted(UNPAIRED)
                                               for k in (0, 1, 3, 7, 9, 12, 15, 16) if k >= UNPAIRED[name][0]])
def test_unpaired_shapes_equal_fixed_blocks(name, waves_per_cu):
    _, make, kw = UNPAIRED[name]
    n = 64 * waves_per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 7
    w = make().with_(n_traj=n)
    print(f"unpaired {name} n={n}", flush=True)
    a, ha = gpu_run(w, **kw)
    b, hb = gpu_run(w, block_size=256, blocks_per_cu=2, **kw)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)
    assert int(ha["count"].sum()) + ha["n_ended_early"] + ha["n_censored"] == n
    np.testing.assert_array_equal(ha["count"], hb["count"])
    assert ha["n_steps_total"] == hb["n_steps_total"]
