"""GPU parity of the FP64 plaquette where the walk along x3 has uneven chunks, a
partial last workgroup, one chunk or two layers, and of the tiles next to it,
against the oracle's plaquette of the same links.  Both sides sum the same
SU(3) matrices in FP64 in different orders and agree to 1e-13.
tests/host/route_check.cpp holds the route of each shape."""
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


@pytest.mark.parametrize("L,nlat,flip", [
    ((6, 10, 14, 630), 1, None),  # 157 chunks of 4 or 5 sites, 131880 threads: a partial last workgroup
    ((6, 10, 14, 318), 2, 0xF),   # 79 chunks of 4 or 5 sites per layer
    ((6, 10, 14, 314), 2, 0xF),   # by tiles
    ((26, 26, 26, 30), 1, None),  # 7 chunks of 4 or 5 sites: more than 4096 tiles
    ((64, 64, 20, 4), 1, None),   # whole columns
    ((64, 64, 18, 4), 1, None),   # by tiles
    ((32, 32, 32, 8), 1, None),   # 65536 threads
    ((24, 24, 24, 16), 2, 0x8),   # two layers, four chunks
])
def test_plaquette_on_either_side_of_the_walk(hb, L, nlat, flip):
    from oracle import su3ref

    print(f"plaquette L={L} nlat={nlat} flip={flip}", flush=True)
    lat = hb.Lattice(L, nlat=nlat, flip_mask=flip, seed=12)
    lat.start(True)
    lat.sweep(1, 5.7)
    got = lat.plaquette()
    ref = su3ref.Oracle(L, nlat=nlat, flip_mask=flip, seed=12)
    ref.set_links(lat.get_links())
    want = ref.plaquette()
    assert np.abs(got - want).max() < 1e-13, (got, want)
    assert lat.plaquette().tobytes() == got.tobytes()
    V = int(np.prod(L))
    bad = lat.get_links()
    bad[[0, 2 * V, 4 * nlat * V - 1], 3] = np.nan
    lat.set_links(bad)
    with pytest.raises(hb.SU3Error) as e:
        lat.plaquette()
    assert e.value.status == hb.su3hb.SU3_ENUMERIC and "3 links" in str(e.value)
