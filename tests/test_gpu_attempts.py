"""GPU tests of measured sweeps with several attempts per subgroup: six waves
per tile of 64 links (lattices of up to 256 tiles in FP64, 512 in FP32) and
three."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hb():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1179_amd as hb_

    return hb_


def _say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("L", [(4, 4, 6, 4), (12, 12, 14, 18), (16, 16, 16, 34), (16, 16, 32, 34)])
@pytest.mark.parametrize("nlat,precision", [(1, 64), (2, 64), (1, 32), (2, 32)])
@pytest.mark.parametrize("nhit,beta", [(2, 0.5), (3, 5.7), (9, 0.5), (64, 0.3)])
def test_measured_sweeps_as_plain_ones(hb, L, nlat, precision, nhit, beta):
    """sweep_measure leaves the links and counters of sweep, bit for bit, and its
    plaquettes are those of su3_plaquette in another order: 1e-13; FP32, whose
    fused sums take FP32 staples, 1e-7."""
    _say(f"measured attempts L={L} nlat={nlat} precision={precision} nhit={nhit} beta={beta}")
    a, b = (hb.Lattice(L, nlat=nlat, precision=precision, nhit=nhit, seed=6) for _ in range(2))
    a.start(True)
    b.start(True)
    fused = a.sweep_measure(2, beta)
    b.sweep(2, beta)
    assert np.array_equal(a.get_links(), b.get_links())
    assert a.counters() == b.counters()
    assert np.abs(fused[1] - b.plaquette()).max() <= (1e-13 if precision == 64 else 1e-7)
