"""Units of work, LDS windows and the library's own launch shape against the plainest
launch: one block size of 128, one block per 128 segments, device atomics only."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _showers(sizes, zenith, dedx):
    out, first = [], 0
    for i, n in enumerate(sizes):
        out.append(W.make_shower(n, seed=400 + i, zenith_deg=zenith, azimuth_deg=37.0 * i, beta="R", dedx=dedx,
                                 core=(40.0 * i, -25.0 * i), first_id=first))
        first += n
    return W.concat_showers(out)


def _run(S, det, ns, cells, dtype):
    bins = torch.zeros(ns * cells, dtype=dtype, device="cuda")
    cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
    cphot.propagate(S, det, bins, None, cnt)
    torch.cuda.synchronize()
    return bins, cnt


# segment counts around a tile of 64, launches that share a tile's rounds, showers that
# begin inside a tile and showers of a few segments each
SIZES = [(1,), (63,), (64,), (65,), (1000,), (30_000,), (40, 3, 1, 500, 77), tuple([5] * 30)]


@pytest.mark.parametrize("transport,zenith,dedx,dtype",
                         [("straight", 0.0, None, "int32"), ("layered", 35.0, None, "int64"),
                          ("table", 35.0, None, "float64"), ("curved", 62.0, (0.1, 2.0), "float64"),
                          ("curved_walk", 62.0, (0.1, 2.0), "int32"), ("surrogate", 60.0, (0.1, 2.0), "int64")])
def test_own_shape_equals_plain_launch(transport, zenith, dedx, dtype):
    """Integer counts: equal bin by bin (the order of the additions does not matter). The
    1000 x 1000 grid gives the axis-shaped window, 40 x 40 the whole grid in LDS."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(transport=transport, spectrum="frank_tamm", seed=9, emission="both" if dedx else "cherenkov")
    if transport == "table":
        kw["table"] = cphot.Table(atm, 2200.0)
    if transport == "surrogate":
        sur = cphot.Surrogate(W.SURROGATE_CURVED_LO, W.SURROGATE_CURVED_HI, max_batch=64, geometry="curved")
        sur.set_params(norm=np.array([*W.SURROGATE_CURVED_LO, *W.SURROGATE_CURVED_HI,
                                      *(2.0 / (np.array(W.SURROGATE_CURVED_HI) - np.array(W.SURROGATE_CURVED_LO))), 0,
                                      0, 0, 0, -1e-5, 1e-5, 1, 1e-5, 1e-5]))
        kw["surrogate"] = sur
    for sizes in SIZES:
        seg, offs, geom = _showers(sizes, zenith, dedx)
        seg, g, off = cphot.upload(seg, geom, offs)
        S = cphot.make_segments(seg, g, off)
        for side in (40, 1000):
            grid = dict(kw, nx=side, ny=side - 3, cell=10.0)
            ref = _run(S, cphot.make_detector(atm, **grid, block_size=128, lds_hist=0), len(sizes), side * (side - 3),
                       getattr(torch, dtype))
            assert int(ref[1][3]) > 0
            for shape in (dict(), dict(lds_hist=1), dict(block_size=256, grid_blocks=3, lds_hist=1, hist_window=9),
                          dict(block_size=512, lds_hist=1, hist_window=30, hist_window_h=12, hist_window_dx=7)):
                if transport == "surrogate" and shape.get("block_size") == 512:
                    continue  # the network's tables leave a block of 512 little LDS
                got = _run(S, cphot.make_detector(atm, **grid, **shape), len(sizes), side * (side - 3),
                           getattr(torch, dtype))
                assert torch.equal(got[0], ref[0]), (sizes, side, shape)
                assert torch.equal(got[1], ref[1]), (sizes, side, shape)


@pytest.mark.parametrize("transport", ["straight", "layered", "curved"])
def test_records_of_shared_tiles(transport):
    """List mode writes every record of its segments once, whatever the units of work: the
    counts of its states equal the propagation's counters."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    for sizes in ((1,), (65,), (300,), (40, 3, 1, 500, 77)):
        seg, offs, geom = _showers(sizes, 50.0, (0.1, 2.0))
        seg, g, off = cphot.upload(seg, geom, offs)
        S = cphot.make_segments(seg, g, off)
        det = cphot.make_detector(atm, transport=transport, spectrum="frank_tamm", seed=4, emission="both", nx=200,
                                  ny=200, cell=10.0)
        counts = torch.zeros(S.n, dtype=torch.int32, device="cuda")
        cphot.segment_counts(S, det, counts)
        ends = torch.cumsum(counts, 0, dtype=torch.int64)
        total = int(ends[-1])
        rec = torch.full((total * cphot.RECORD_BYTES,), 255, dtype=torch.uint8, device="cuda")
        cphot.trace_records(S, det, ends - counts, rec)
        r = cphot.records_to_numpy(rec.cpu())
        n = counts.cpu().numpy()
        assert np.array_equal(r["seg"], np.repeat(np.arange(S.n, dtype=np.uint64), n))
        assert np.array_equal(r["k"], np.concatenate([np.arange(x) for x in n]))
        _, cnt = _run(S, det, len(sizes), 200 * 200, torch.int32)
        cnt = cnt.cpu().numpy()
        states = np.bincount(r["state"], minlength=4)
        assert cnt[3] == total and cnt[4] == states[1] and cnt[5] == states[2]
        assert cnt[6] == states[3] and cnt[7] == states[0]


@pytest.mark.parametrize("transport,detector,bunch", [("straight", "grid", 1), ("curved", "grid", 1),
                                                      ("layered", "spheres", 5)])
@pytest.mark.parametrize("sizes", [(70_001,), (20_000, 64, 5, 30_000)])
def test_more_blocks_than_fit(transport, detector, bunch, sizes):
    """Blocks' ranges that fall with the block index, and runs whose last units are halved:
    every record once, whatever the number of blocks."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(transport=transport, spectrum="frank_tamm", seed=9, bunch=bunch, detector=detector)
    kw.update(dict(nx=100, ny=100, cell=10.0) if detector == "grid" else dict(snx=10, sny=10, pitch=150.0, radius=6.0))
    seg, offs, geom = _showers(sizes, 50.0, None)
    S = cphot.make_segments(*cphot.upload(seg, geom, offs))
    cells = 10_000 if detector == "grid" else 100
    ref = _run(S, cphot.make_detector(atm, **kw, block_size=128, lds_hist=0), len(sizes), cells, torch.int64)
    for block in (128, 256, 512):
        for blocks in (1, 7, 1000, 2100, 10**6):
            got = _run(S, cphot.make_detector(atm, **kw, block_size=block, grid_blocks=blocks, lds_hist=1), len(sizes),
                       cells, torch.int64)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]), (block, blocks)


@pytest.mark.parametrize("transport", ["straight", "layered", "table", "surrogate"])
@pytest.mark.parametrize("side", [10, 250])
def test_own_shape_on_spheres(transport, side):
    """Sphere and time counts: an array that fits in LDS and one of 62,500 spheres, which
    does not; integer counts, equal in every bin."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(transport=transport, spectrum="frank_tamm", seed=9, bunch=2, detector="spheres", snx=side, sny=side,
              pitch=1500.0 / side, radius=300.0 / side, n_t=64, dt=2.0)
    if transport == "table":
        kw["table"] = cphot.Table(atm, 2200.0)
    if transport == "surrogate":
        lo, hi = np.array(W.SURROGATE_LO), np.array(W.SURROGATE_HI)
        kw["surrogate"] = cphot.Surrogate(lo, hi, max_batch=64)
        kw["surrogate"].set_params(norm=np.array([*lo, *hi, *(2.0 / (hi - lo)), 0, 0, 0, 0, -1e-5, 1e-5, 1, 1e-5, 1e-5]))
    for sizes in ((1,), (65,), (20_000,), (40, 3, 1, 500, 77)):
        seg, offs, geom = _showers(sizes, 30.0, None)
        S = cphot.make_segments(*cphot.upload(seg, geom, offs))
        out = []
        for shape in (dict(), dict(block_size=128, lds_hist=0)):
            bins = torch.zeros(len(sizes) * side * side, dtype=torch.int64, device="cuda")
            times = torch.zeros(len(sizes) * side * side * 65, dtype=torch.int32, device="cuda")
            cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
            cphot.propagate(S, cphot.make_detector(atm, **kw, **shape), bins, times, cnt)
            out.append((bins, times, cnt))
        assert all(torch.equal(a, b) for a, b in zip(*out)), sizes
        assert len(sizes) == 1 or int(out[0][2][7]) > 0
