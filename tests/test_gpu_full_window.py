"""Blocks that count hundreds of millions of records in one window."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _segments(n, charge):
    sh = W.make_shower(n, seed=3, xmax=500.0, zenith_deg=0.0, beta="R")
    seg = {k: v.copy() for k, v in sh.seg.items()}
    seg["charge"][:] = charge
    seg, geom, _ = cphot.upload(seg, np.array([[*sh.core, *sh.axis]]), None)
    return cphot.make_segments(seg, geom)


def _run(S, **shape):
    atm = cphot.Atmosphere(**cases.ATMO_STRAIGHT)
    det = cphot.make_detector(atm, transport="straight", detector="grid", nx=1000, ny=1000, cell=10.0, seed=9, **shape)
    bins = torch.zeros(1000 * 1000, dtype=torch.int64, device="cuda")
    cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    cphot.propagate(S, det, bins, None, cnt)
    b.record()
    torch.cuda.synchronize()
    return bins, cnt, a.elapsed_time(b)


def test_window_counts_the_units_own_records():
    """Eight blocks with about 2.7e8 records each, an eighth of what a window may count, from
    segments of some 5e5 that sixteen units share: at the rate of a launch an eighth as long
    (4.3 records per ns in the window, 1.2 with device atomics; at least 0.7 of it, a launch's
    uneven end being within a tenth), and the counts of device atomics alone."""
    shape = dict(block_size=512, grid_blocks=8)
    few = _segments(512, 90.0)
    _run(few, lds_hist=1, **shape)
    _, cnt, ms = _run(few, lds_hist=1, **shape)
    rate_few = int(cnt[3]) / ms
    many = _segments(4096, 90.0)
    bins, cnt, ms = _run(many, lds_hist=1, **shape)
    assert int(cnt[3]) > 2e9
    ref, ref_cnt, _ = _run(many, lds_hist=0)
    assert torch.equal(bins, ref) and torch.equal(cnt, ref_cnt)
    assert int(cnt[3]) / ms > 0.7 * rate_few, (int(cnt[3]) / ms, rate_few)
