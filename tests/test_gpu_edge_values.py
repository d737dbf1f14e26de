"""GPU tests of links and couplings at the ends of the floating-point range:
rows whose squared norm is 0 or overflows, NaN rows, and couplings so large
that projections of twice the size would overflow.  The library treats them as
the plain arithmetic of the FP64 oracle does."""
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


def _same(got, want, tol):
    """Equal where not finite, within tol elsewhere."""
    f = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), f)
    assert np.array_equal(got[~f], want[~f], equal_nan=True)
    assert np.abs(got[f] - want[f]).max() < tol


def test_reunitarise_rows_of_any_norm(hb):
    """A row whose squared norm overflows becomes 0, one whose squared norm is
    0 becomes inf or NaN by the sign of each entry; other rows and links are
    as usual.  Rows 0 and 1, which are stored."""
    from oracle import su3ref

    ref = su3ref.Oracle((4, 4, 4, 4), seed=8)
    ref.start(True)
    links = ref.links().copy()
    for k, (lo, hi, f) in enumerate([(0, 6, 1e160), (6, 12, 1e160), (0, 6, 1e-200), (0, 6, 0.0), (6, 12, 0.0),
                                     (0, 6, 1e-155), (0, 12, 1e-150), (0, 12, 1e150)]):
        links[4 * k + 3, lo:hi] *= f
    links[101, 0] = np.inf
    links[105, 8] = np.nan
    lat = hb.Lattice((4, 4, 4, 4), seed=8)
    lat.set_links(links)
    ref.set_links(links)
    lat.reunitarise()
    ref.reunitarise()
    # 1e-155: the squared norm is subnormal, 1e-310 with 2^-1074 the last place, and so the norm off by up to 1e-14
    _same(lat.get_links()[:, :12], ref.links()[:, :12], 1e-13)


@pytest.mark.parametrize("nlat,nhit", [(1, 1), (1, 3), (2, 1)])
@pytest.mark.parametrize("precision", [64, 32])
def test_a_nan_row_stays_in_its_row(hb, nlat, nhit, precision):
    """A link with a NaN in its row 1 gets no update: its projections are NaN,
    every attempt is rejected, and row 0 stays as it was; its neighbours'
    staples are NaN, and they stay too.  Links and counters as the oracle's,
    FP32 links within the rounding of a sweep where they hold no update."""
    from oracle import su3ref

    L = (4, 4, 4, 6)
    ref = su3ref.Oracle(L, nlat=nlat, flip_mask=7 if nlat == 2 else None, nhit=nhit, seed=5)
    ref.start(True)
    links = ref.links().copy()
    links[17, 6:18] = np.nan  # row 2 is rebuilt from rows 0 and 1
    lat = hb.Lattice(L, nlat=nlat, precision=precision, nhit=nhit, seed=5)
    lat.set_links(links)
    ref.set_links(links)
    lat.sweep(1, 5.7)
    ref.sweep(1, 5.7)
    got, want = lat.get_links()[:, :12], ref.links()[:, :12]
    assert np.isfinite(want[17, :6]).all() and np.isnan(want[17, 6:]).all()
    if precision == 64:
        _same(got, want, 1e-12)
        assert lat.counters()[1:] == ref.counters()
    else:
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.abs(got[17, :6] - want[17, :6]).max() < 1e-6


@pytest.mark.parametrize("precision,beta", [(64, 1.5e153), (32, 2e18)])
@pytest.mark.parametrize("nhit", [1, 2])
def test_layer_couplings_near_the_overflow(hb, precision, beta, nhit):
    """A cold double-layered torus: every staple is 6 beta, whose square is
    finite; that of 12 beta is not.  Every attempt is accepted, as the oracle's."""
    from oracle import su3ref

    L = (4, 4, 4, 4)
    lat = hb.Lattice(L, nlat=2, precision=precision, nhit=nhit, seed=8)
    ref = su3ref.Oracle(L, nlat=2, flip_mask=7, nhit=nhit, seed=8)
    lat.start(False)
    ref.start(False)
    lat.sweep_betas(1, beta, beta)
    ref.sweep_betas(1, beta, beta)
    assert lat.counters()[1:] == ref.counters()
    assert ref.counters()[0] == ref.counters()[1]
    _same(lat.get_links(), ref.links(), 1e-12 if precision == 64 else 1e-6)
