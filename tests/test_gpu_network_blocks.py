"""The network's transports in blocks of 512 with LDS counts (63 KB of tables beside them)."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


@pytest.mark.parametrize("geometry", ["planar", "curved"])
@pytest.mark.parametrize("side", [40, 1000])
def test_counts_equal_plain_launch(geometry, side):
    """A grid that fits, a window of one that does not, a caller's window off the centre: the
    counts of device atomics alone, over one segment, a tile and one more, and many."""
    curved = geometry == "curved"
    lo, hi = (W.SURROGATE_CURVED_LO, W.SURROGATE_CURVED_HI) if curved else (W.SURROGATE_LO, W.SURROGATE_HI)
    sur = cphot.Surrogate(lo, hi, max_batch=64, geometry=geometry)
    sur.set_params(norm=np.array([*lo, *hi, *(2.0 / (np.array(hi) - np.array(lo))), 0, 0, 0, 0, -1e-5, 1e-5, 1, 1e-5, 1e-5]))
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(transport="surrogate", surrogate=sur, spectrum="frank_tamm", seed=9, emission="both", nx=side, ny=side - 3,
              cell=10.0)
    for n in (1, 65, 30_000):
        sh = W.make_shower(n, seed=3, zenith_deg=60.0 if curved else 35.0, azimuth_deg=15.0, beta="R", dedx=(0.1, 2.0))
        seg, geom, _ = cphot.upload(sh.seg, np.array([[*sh.core, *sh.axis]]), None)
        S, out = cphot.make_segments(seg, geom), []
        for shape in (dict(block_size=128, lds_hist=0), dict(block_size=512, lds_hist=1),
                      dict(block_size=512, lds_hist=1, hist_window=30, hist_window_h=12, hist_window_dx=7)):
            bins = torch.zeros(side * (side - 3), dtype=torch.int64, device="cuda")
            cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
            cphot.propagate(S, cphot.make_detector(atm, **kw, **shape), bins, None, cnt)
            out.append((bins, cnt))
        assert int(out[0][1][3]) > 0
        assert all(torch.equal(a, b) for o in out[1:] for a, b in zip(o, out[0])), n
