"""The caller's window shift with the library's own launch shape."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _time(run):
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("lds", [-1, 1])
@pytest.mark.parametrize("along", ["x", "y"])
def test_window_follows_the_shift(along, lds):
    """A shower 3.5 km from the grid's centre puts its light into few cells there. With a
    window around them the device atomics, one a photon onto those cells and most of the
    time, are gone: at most half the time of the centred window. Shifts beyond the grid end
    at its edge; the bins are the same always."""
    atm = cphot.Atmosphere(**cases.ATMO_STRAIGHT)
    sh = W.make_shower(100_000, seed=3, xmax=500.0, zenith_deg=0.0, beta="R")
    seg = {k: v.copy() for k, v in sh.seg.items()}
    for k in (along + "0", along + "1"):
        seg[k] += np.float32(3500.0)
    seg, geom, _ = cphot.upload(seg, np.array([[*sh.core, *sh.axis]]), None)
    S = cphot.make_segments(seg, geom)
    bins = torch.zeros(1000 * 1000, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
    times, ref = {}, None
    for shift in (0, 350, 10**9, -10**9, 2**31 - 1, -2**31):
        kw = {"hist_window_d" + along: shift}
        det = cphot.make_detector(atm, transport="straight", detector="grid", nx=1000, ny=1000, cell=10.0, seed=9,
                                  lds_hist=lds, **kw)
        bins.zero_()
        cnt.zero_()
        cphot.propagate(S, det, bins, None, cnt)
        torch.cuda.synchronize()
        if ref is None:
            ref = (bins.clone(), cnt.clone())
            assert int(cnt[7]) > 1_000_000
        assert torch.equal(bins, ref[0]) and torch.equal(cnt, ref[1]), shift
        if shift in (0, 350):
            times[shift] = _time(lambda: cphot.propagate(S, det, bins, None, cnt))
    assert times[350] < 0.5 * times[0], times
