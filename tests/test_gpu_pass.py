"""GPU tests of the pass kernels where their own branches can go wrong: link
offsets of 64 bits, the search for a tile's job in a batch, and the FP32
staple terms kept apart for per-layer couplings."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def hb():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_0904_1179_amd as hb_

    return hb_


def _say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("L,nlat,precision,kind", [
    ((96, 96, 98, 100), 1, 64, "measure"),  # 45.2e6 links per block, 96 bytes each: just over 4 GiB
    ((80, 80, 84, 84), 2, 64, "betas"),
    ((96, 96, 98, 100), 2, 32, "measure"),  # 90.3e6 links of 48 bytes
])
def test_blocks_over_4_gib(hb, L, nlat, precision, kind):
    """Sampled links after one sweep against the oracle, computed link by link;
    the fused plaquette against su3_plaquette."""
    import torch
    from cone import FirstSweepCone, sample_lids
    from oracle import su3ref

    link_bytes, _ = hb.su3_footprint(hb.make_params(L, nlat=nlat, precision=precision))
    assert link_bytes // 8 > 1 << 32
    if torch.cuda.mem_get_info()[0] < link_bytes + (2 << 30):
        pytest.skip("not enough device memory")
    _say(f"64-bit offsets L={L} nlat={nlat} precision={precision} {kind}")
    lat = hb.Lattice(L, nlat=nlat, precision=precision, seed=1)
    lat.start(True)
    if kind == "betas":
        lat.sweep_betas(1, 5.7, 5.7)  # equal couplings: the single-coupling chain
    else:
        fused = lat.sweep_measure(1, 5.7)[0]
        # FP32: the fused sum takes its staples in FP32, rounded at random
        assert np.abs(fused - lat.plaquette()).max() <= (1e-13 if precision == 64 else 1e-7)
    lids = sample_lids(4 * lat.V * nlat, 18)
    got = lat.link_sample(lids)
    cone = FirstSweepCone(L, nlat=nlat, seed=1, beta=5.7)
    dev = np.array([np.abs(su3ref.to_complex(got[k]) - cone.value(l)).max() for k, l in enumerate(lids)])
    if precision == 64:
        assert dev.max() < 1e-12
    else:
        assert np.median(dev) < 1e-5 and np.mean(dev < 1e-4) > 0.9
    assert lat.counters()[1] == 12 * lat.V * nlat


@pytest.mark.parametrize("njobs", [1, 2, 63, 64, 65, 130, 200])
def test_every_tile_finds_its_job(hb, njobs):
    """Batches around the 64 jobs a wave looks at in one step, of lattices of one
    to four tiles with a partial last tile: every job as if alone, bit for bit."""
    from paper_0904_1179_amd import serve

    shapes = [(2, 2, 2, 2), (4, 2, 4, 2), (4, 4, 4, 2), (6, 4, 4, 4), (4, 4, 6, 2)]
    srv = serve.Server(arena_bytes=256 << 20, max_active=256)
    ids = [srv.submit(serve.make_job(shapes[k % 5], 5.7, 2, seed=k + 1, precision=64)) for k in range(njobs)]
    while True:
        active, queued, _ = srv.run(4)
        if not active and not queued:
            break
    for k, jid in enumerate(ids):
        r = srv.poll(jid)
        lat = hb.Lattice(shapes[k % 5], seed=k + 1)
        lat.start(True)
        lat.sweep(2, 5.7)
        assert np.array_equal(np.array(r["plaquette"][:2]), lat.plaquette()), k
        assert (r["kp_attempts"], r["kp_accepts"]) == lat.counters()[1:], k


@pytest.mark.parametrize("L,flip,nhit", [((4, 4, 4, 6), 0x7, 1), ((6, 4, 10, 2), 0xF, 2), ((2, 2, 2, 2), 0x5, 1)])
def test_fp32_layer_couplings_against_oracle(hb, L, flip, nhit):
    """FP32 links with one coupling per layer against the FP64 oracle, one
    sweep: about a hundred roundings of 6e-8 a link, carried through eight
    passes, so 1e-5 on the median and 1e-4 where no accept decision differs."""
    from oracle import su3ref

    _say(f"fp32 betas L={L} flip={flip} nhit={nhit}")
    lat = hb.Lattice(L, nlat=2, flip_mask=flip, precision=32, nhit=nhit, seed=3)
    lat.start(True)
    lat.sweep_betas(1, 5.5, 6.2)
    ref = su3ref.Oracle(L, nlat=2, flip_mask=flip, nhit=nhit, seed=3)
    ref.start(True)
    ref.sweep_betas(1, 5.5, 6.2)
    d = np.abs(lat.get_links() - ref.links()).max(axis=1)
    assert np.median(d) < 1e-5 and np.mean(d < 1e-4) > 0.9
    if nhit == 1:
        assert lat.counters()[1] == ref.counters()[0]


@pytest.mark.parametrize("nhit", [1, 2, 4])
@pytest.mark.parametrize("nlat,precision", [(1, 64), (2, 64), (1, 32), (2, 32)])
@pytest.mark.parametrize("beta", [0.4, 5.7])  # 0.4: many links miss outside the draws made ahead
def test_three_waves_per_tile_as_six(hb, nhit, nlat, precision, beta):
    """Small batches run six waves per tile of 64 links, large ones three; both
    make the same draws and sums in the same order, so each job's plaquettes
    and counts have the same bits in a batch of more than 768 tiles as alone."""
    from paper_0904_1179_amd import serve

    _say(f"three waves nhit={nhit} nlat={nlat} precision={precision} beta={beta}")
    L = (4, 6, 6, 38)  # 2736 links per pass and layer: 42.75 tiles
    tiles = -(-nlat * 2736 // 64)
    njobs = 768 // tiles + 1
    srv = serve.Server(arena_bytes=512 << 20, max_active=64)
    ids = [srv.submit(serve.make_job(L, beta, 2, seed=k + 1, precision=precision, nlat=nlat, nhit=nhit))
           for k in range(njobs)]
    while True:
        nactive, nqueued, _ = srv.run(2)
        if nactive == 0 and nqueued == 0:
            break
    for k in {0, njobs // 2, njobs - 1}:
        r = srv.poll(ids[k])
        lat = hb.Lattice(L, nlat=nlat, precision=precision, seed=k + 1, nhit=nhit)
        lat.start(True)
        lat.sweep(2, beta)
        assert np.array_equal(np.array(r["plaquette"][:1 + nlat]), lat.plaquette())
        assert (r["kp_attempts"], r["kp_accepts"]) == lat.counters()[1:]


@pytest.mark.parametrize("L,nlat,flip,precision", [
    ((2, 2, 2, 2), 1, None, 64),          # 8 of the 64 half-indices of a tile
    ((4, 4, 4, 2), 2, 0xF, 64),           # exactly one tile
    ((6, 4, 10, 2), 2, 0x5, 32),          # 240: a partial last tile
    ((66, 4, 2, 4), 1, None, 64),         # 1056
    ((32, 32, 32, 12), 1, None, 64),      # 98304 columns and chunks: tiles
    ((32, 32, 32, 16), 1, None, 64),      # 131072: the walk
])
def test_plaquette_tiles_and_walk(hb, L, nlat, flip, precision):
    """Hot lattices against the oracle.  Each of the terms, at most 1 in
    magnitude, takes some 60 roundings of 1.1e-16, and the partial sums of a
    hot lattice stay small: below 1e-13.  FP32 holds links rounded to 6e-8,
    whose errors average out over the plaquettes: below 1e-7."""
    from oracle import su3ref

    _say(f"plaquette L={L} nlat={nlat} flip={flip} precision={precision}")
    lat = hb.Lattice(L, nlat=nlat, flip_mask=flip, precision=precision, seed=9)
    ref = su3ref.Oracle(L, nlat=nlat, flip_mask=flip, seed=9)
    lat.start(True)
    ref.start(True)
    assert np.abs(lat.plaquette() - ref.plaquette()).max() < (1e-13 if precision == 64 else 1e-7)
