"""The classical trajectory of the matched and time-node tables ends 200 e-folds after its start, whatever
strides reach that time: a node beyond is refused (time nodes) or keeps the Bunch-Davies noise (phi nodes),
as in the oracle's sequential solve.  Tolerances: the tables' parity bars."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
from paper_2410_13683_amd import fpt  # noqa: E402

# slow roll on a nearly flat potential: phi falls by 0.198 in 200 e-folds
POT = (0, 1.0, -9.0, 1e-3, 1e-3)
START = (1.0, -1e-3)
REF = 0.999999                    # passed 1e-3 e-folds after the start


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _pot():
    return fpt.make_potential(*POT, 3.0, 0.0, -1.0)


@pytest.mark.parametrize("t", [199.9, 199.998, 200.0, 200.03, 200.08, 200.2])
def test_time_nodes_beyond_the_end_are_refused(t):
    print(f"time node {t}", flush=True)
    beyond = t + 1e-3 > 200.0
    args = (1, t, t, *START, REF)
    for gpu, cpu, sigma in ((fpt.fpt_noise_table_matched_time, orc.noise_table_matched_time, 1.0),
                            (fpt.fpt_noise_table_bessel2d_time, orc.noise_table_bessel2d_time, 0.1)):
        if beyond:
            with pytest.raises(ValueError):
                cpu(*POT, sigma, *args)
            with pytest.raises(fpt.FptError):
                gpu(_pot(), sigma, *args)
            continue
        g, o = gpu(_pot(), sigma, *args), cpu(*POT, sigma, *args)
        np.testing.assert_allclose(g[0], o[0], rtol=1e-9, atol=0)
        np.testing.assert_allclose(g[3], o[3], rtol=1e-9, atol=0)


def test_phi_nodes_beyond_the_end_keep_their_noise():
    """Nodes passed at N = 199.92 .. 200.08: those after N = 200 are never reached."""
    phi = orc.noise_table_matched_time(*POT, 1.0, 2, 199.92, 199.99, *START, REF)[3]
    slope = (phi[1] - phi[0]) / 0.07
    lo, hi = phi[1] + 0.09 * slope, phi[0]
    print(f"phi nodes {lo} {hi}", flush=True)
    o = orc.noise_table_matched(*POT, 1.0, 17, lo, hi, *START)
    g = fpt.fpt_noise_table_matched(_pot(), 1.0, 17, lo, hi, *START)
    assert 4 < int(np.sum(o[2] == 1.0)) < 13
    np.testing.assert_array_equal(g[2] == 1.0, o[2] == 1.0)
    np.testing.assert_allclose(g[2], o[2], rtol=1e-9, atol=0)
