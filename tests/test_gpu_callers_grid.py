"""Launches whose grid the caller gives, smaller than the chip."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _launch(n, **shape):
    sh = W.make_shower(n, seed=3, xmax=500.0, zenith_deg=20.0, azimuth_deg=15.0, beta="R")
    seg, geom, _ = cphot.upload(sh.seg, np.array([[*sh.core, *sh.axis]]), None)
    S = cphot.make_segments(seg, geom)
    det = cphot.make_detector(cphot.Atmosphere(**cases.ATMO_STRAIGHT), transport="straight", spectrum="frank_tamm", seed=9,
                              counts="poisson", bunch=2, nx=100, ny=60, cell=10.0, **shape)
    bins = torch.zeros(6000, dtype=torch.int64, device="cuda")
    cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
    return lambda: cphot.propagate(S, det, bins, None, cnt), bins, cnt


def _time(run):
    best = 1e9
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 5)
    return best


def test_tiles_are_shared_by_the_waves_there_are():
    """5,000 segments on 7 blocks against 180,000 on 252: as many a block, each block alone on
    its CU, so the times are near. Tiles shared by sixteen units, as the whole chip's waves
    would need them, repeat the Poisson set-up for nothing: 2.9 times as long."""
    times = [_time(_launch(n, block_size=256, grid_blocks=g, lds_hist=1)[0]) for n, g in ((5_000, 7), (180_000, 252))]
    assert times[0] < 1.4 * times[1], times


@pytest.mark.parametrize("blocks", [1, 3, 40, 5000])
def test_counts_do_not_depend_on_the_grid(blocks):
    ref = _launch(9_000, block_size=128, lds_hist=0)
    ref[0]()
    for block in (128, 256, 512):
        for lds in (0, 1):
            run, bins, cnt = _launch(9_000, block_size=block, grid_blocks=blocks, lds_hist=lds)
            run()
            assert torch.equal(bins, ref[1]) and torch.equal(cnt, ref[2]), (block, lds)
