"""GPU tests of several attempts per subgroup on every route: six waves per
tile of 64 links (lattices of up to 256 tiles in FP64, 512 in FP32), three, and
one (most attempts miss, or large lattices); measured, plain and with per-layer
couplings; with few lanes of a wave missing and with nearly all."""
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


@pytest.mark.parametrize("L,nlat,flip,nhit,beta,kind", [
    ((4, 4, 6, 4), 1, None, 3, 0.5, "sweep"),        # six waves
    ((2, 2, 2, 2), 1, None, 64, 0.2, "sweep"),       # one wave, 8 of its 64 lanes hold links
    ((6, 4, 10, 2), 2, 0x5, 64, 0.5, "betas"),       # one wave, a partial last tile
    ((8, 8, 8, 8), 1, None, 17, 2.0, "sweep"),       # one wave: rounds that end at the last attempt
    ((12, 12, 14, 18), 1, None, 3, 4.2, "sweep"),    # 284 tiles: three waves
    ((12, 12, 14, 18), 1, None, 7, 0.5, "measure"),  # one wave
    ((16, 16, 16, 34), 1, None, 2, 0.5, "sweep"),    # 1088 tiles: one wave
    ((16, 16, 8, 34), 2, 0xF, 3, 2.0, "measure"),    # 1088 tiles: one wave, two layers
    ((12, 12, 12, 12), 2, 0x7, 3, 5.5, "betas"),     # 324 tiles: three waves
    ((16, 16, 8, 34), 2, 0x7, 2, 5.5, "betas"),      # 1088 tiles: one wave
])
def test_attempts_against_oracle(hb, L, nlat, flip, nhit, beta, kind):
    """One sweep, FP64: counters exactly, and every link to the rounding of some
    hundred operations (1e-14) times the factor by which the oracle's own
    links answer a change of the start links, which is large where staples
    are small (measured here with a change of 1e-13)."""
    from oracle import su3ref

    _say(f"attempts L={L} nlat={nlat} flip={flip} nhit={nhit} beta={beta} {kind}")
    lat = hb.Lattice(L, nlat=nlat, flip_mask=flip, nhit=nhit, seed=13)
    ref = su3ref.Oracle(L, nlat=nlat, flip_mask=flip, nhit=nhit, seed=13)
    lat.start(True)
    ref.start(True)
    start = ref.links().copy()

    def run(o):
        if kind == "betas":
            o.sweep_betas(1, beta, beta + 0.4)
        else:
            o.sweep(1, beta)
        return o.links().copy()

    want, counts, plaq = run(ref), ref.counters(), ref.plaquette()
    moved = su3ref.Oracle(L, nlat=nlat, flip_mask=flip, nhit=nhit, seed=13)
    moved.start(True)
    moved.set_links(start + 1e-13 * np.random.default_rng(1).normal(size=start.shape))
    moved.reunitarise()
    answer = np.abs(run(moved) - want).max() / 1e-13
    if kind == "measure":
        fused = lat.sweep_measure(1, beta)[0]
        assert np.abs(fused - plaq).max() < max(1e-13, 1e-14 * answer)
    elif kind == "betas":
        lat.sweep_betas(1, beta, beta + 0.4)
    else:
        lat.sweep(1, beta)
    dev = np.abs(lat.get_links() - want).max()
    _say(f"  max |dU| {dev:.2e}, bound {max(1e-12, 1e-14 * answer):.2e}")
    assert dev < max(1e-12, 1e-14 * answer)
    assert lat.counters()[1:] == counts


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


@pytest.mark.parametrize("nhit,beta,tiles", [(9, 0.4, 600), (2, 0.4, 2100), (5, 2.0, 2100)])
@pytest.mark.parametrize("nlat,precision", [(1, 64), (2, 64), (1, 32), (2, 32)])
def test_one_wave_per_tile_as_six(hb, nhit, beta, tiles, nlat, precision):
    """Jobs in a batch large enough for one wave per tile against the same
    lattices alone, which run six (or three): the same draws and sums in the
    same order, so the same bits of the plaquettes, and the same counts."""
    from paper_0904_1179_amd import serve

    _say(f"one wave nhit={nhit} beta={beta} nlat={nlat} precision={precision}")
    L = (4, 6, 10, 38)  # 4560 links per pass and layer: 71.25 tiles
    njobs = tiles // -(-nlat * 4560 // 64) + 1
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


@pytest.mark.parametrize("L", [(2, 2, 2, 2), (12, 12, 14, 18), (16, 16, 32, 34)])
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("nhit,beta", [(3, 5.7), (20, 1.0)])
def test_equal_layer_couplings_as_one(hb, L, precision, nhit, beta):
    """With both couplings equal to beta the weighted staple is beta times the
    plain one up to rounding: counters differ in at most one decision in ten
    thousand, and in FP64 not at all on these lattices."""
    _say(f"equal couplings L={L} precision={precision} nhit={nhit} beta={beta}")
    a, b = (hb.Lattice(L, nlat=2, precision=precision, nhit=nhit, seed=2) for _ in range(2))
    a.start(True)
    b.start(True)
    a.sweep_betas(1, beta, beta)
    b.sweep(1, beta)
    if precision == 64:
        assert a.counters() == b.counters()
    else:
        assert abs(a.counters()[1] - b.counters()[1]) <= 1e-4 * b.counters()[1]
    d = np.abs(a.get_links() - b.get_links()).max(axis=1)
    assert np.median(d) < (1e-13 if precision == 64 else 1e-5)


@pytest.mark.parametrize("L,nlat,precision,kind", [
    ((96, 96, 98, 100), 1, 64, "measure"),  # 45.2e6 links per block, 96 bytes each: just over 4 GiB
    ((80, 80, 84, 84), 2, 64, "betas"),
    ((96, 96, 98, 100), 2, 32, "measure"),  # 90.3e6 links of 48 bytes
])
def test_attempts_in_blocks_over_4_gib(hb, L, nlat, precision, kind):
    """Link offsets of 64 bits with two attempts (one wave per tile): sampled
    links after one sweep against the oracle, computed link by link; the fused
    plaquette against su3_plaquette.  Bounds as for one attempt at this coupling."""
    import os
    import sys

    import torch

    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    from cone import FirstSweepCone, sample_lids
    from oracle import su3ref

    link_bytes, _ = hb.su3_footprint(hb.make_params(L, nlat=nlat, precision=precision))
    assert link_bytes // 8 > 1 << 32
    if torch.cuda.mem_get_info()[0] < link_bytes + (2 << 30):
        pytest.skip("not enough device memory")
    _say(f"attempts, 64-bit offsets L={L} nlat={nlat} precision={precision} {kind}")
    lat = hb.Lattice(L, nlat=nlat, precision=precision, nhit=2, seed=1)
    lat.start(True)
    if kind == "betas":
        lat.sweep_betas(1, 5.7, 5.7)  # equal couplings: the single-coupling chain
    else:
        fused = lat.sweep_measure(1, 5.7)[0]
        assert np.abs(fused - lat.plaquette()).max() <= (1e-13 if precision == 64 else 1e-7)
    lids = sample_lids(4 * lat.V * nlat, 18)
    got = lat.link_sample(lids)
    cone = FirstSweepCone(L, nlat=nlat, seed=1, beta=5.7, nhit=2)
    dev = np.array([np.abs(su3ref.to_complex(got[k]) - cone.value(l)).max() for k, l in enumerate(lids)])
    if precision == 64:
        assert dev.max() < 1e-12
    else:
        assert np.median(dev) < 1e-5 and np.mean(dev < 1e-4) > 0.9
