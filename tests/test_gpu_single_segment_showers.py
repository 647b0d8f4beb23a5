"""Tiles that hold many showers of a segment or a few."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _batch(sizes, zenith=20.0, dedx=None):
    out, first = [], 0
    for i, n in enumerate(sizes):
        out.append(W.make_shower(n, seed=100 + i, xmax=500.0, zenith_deg=zenith, azimuth_deg=37.0 * i, beta="R",
                                 dedx=dedx, core=(20.0 * (i % 7), 0.0), first_id=first))
        first += n
    seg, off, geom = W.concat_showers(out)
    seg, geom, off = cphot.upload(seg, geom, off)
    return cphot.make_segments(seg, geom, off)


def _outputs(ns):
    return (torch.zeros(ns * 10_000, dtype=torch.int32, device="cuda"), None,
            torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda"))


GRID = dict(detector="grid", nx=100, ny=100, cell=10.0)


def _time(run):
    best = 1e9
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 10)
    return best


def test_showers_of_one_segment_are_spread():
    """100 showers of a segment each against one of 100 segments: the same photons, a round
    or less of 64 for each shower instead of full ones, and 100 grids. 2.3 times as long with
    the rounds spread over the units of a tile; seven times where one of them does all."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    det = cphot.make_detector(atm, transport="layered", spectrum="frank_tamm", seed=9, **GRID)
    times = []
    for sizes in ([100], [1] * 100):
        S, out = _batch(sizes), _outputs(len(sizes))
        times.append(_time(lambda: cphot.propagate(S, det, *out)))
    assert times[1] < 4.0 * times[0], times


@pytest.mark.parametrize("transport,zenith,dedx", [("straight", 20.0, (0.1, 2.0)), ("layered", 35.0, None),
                                                   ("table", 35.0, None), ("curved", 62.0, (0.1, 2.0)),
                                                   ("surrogate", 60.0, (0.1, 2.0))])
@pytest.mark.parametrize("sizes", [(1,) * 200, (1, 2, 3) * 40, (1,) * 70 + (5000,) + (2,) * 70])
def test_every_share_once(transport, zenith, dedx, sizes):
    """Each shower's rounds fall to its tile's units once, the last ones of a run in halves
    among them: every record is generated, and the counts are those of one block of 128 with
    device atomics."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(GRID, transport=transport, spectrum="frank_tamm", seed=9, emission="both" if dedx else "cherenkov")
    if transport == "table":
        kw["table"] = cphot.Table(atm, 2200.0)
    if transport == "surrogate":
        lo, hi = np.array(W.SURROGATE_CURVED_LO), np.array(W.SURROGATE_CURVED_HI)
        kw["surrogate"] = cphot.Surrogate(lo, hi, max_batch=64, geometry="curved")
        kw["surrogate"].set_params(norm=np.array([*lo, *hi, *(2.0 / (hi - lo)), 0, 0, 0, 0, -1e-5, 1e-5, 1, 1e-5, 1e-5]))
    S, got = _batch(sizes, zenith, dedx), []
    counts = torch.zeros(S.n, dtype=torch.int32, device="cuda")
    for shape in (dict(block_size=128, grid_blocks=1, lds_hist=0), dict(), dict(block_size=512, grid_blocks=3, lds_hist=1),
                  dict(block_size=256, lds_hist=0)):
        det, out = cphot.make_detector(atm, **kw, **shape), _outputs(len(sizes))
        cphot.propagate(S, det, *out)
        got.append(out)
    cphot.segment_counts(S, det, counts)
    for out in got:
        assert int(out[2][3]) == int(counts.sum()) > 0  # every record once
        assert torch.equal(out[0], got[0][0]) and torch.equal(out[2], got[0][2])
