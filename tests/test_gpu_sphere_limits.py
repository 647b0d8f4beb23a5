"""Sphere arrays in LDS at explicit block sizes, near the largest that a block can hold."""
import numpy as np
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _detector(transport, side, n_t=0, **shape):
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    kw = dict(transport=transport, spectrum="frank_tamm", seed=9, bunch=5, detector="spheres", snx=side, sny=side,
              pitch=1500.0 / side, radius=200.0 / side, n_t=n_t, dt=2.0)
    if transport == "table":
        kw["table"] = cphot.Table(atm, 2200.0)
    if transport == "surrogate":
        lo, hi = np.array(W.SURROGATE_LO), np.array(W.SURROGATE_HI)
        kw["surrogate"] = cphot.Surrogate(lo, hi, max_batch=64)
        kw["surrogate"].set_params(norm=np.array([*lo, *hi, *(2.0 / (hi - lo)), 0, 0, 0, 0, -1e-5, 1e-5, 1, 1e-5, 1e-5]))
    return cphot.make_detector(atm, **kw, **shape)


def _segments(n):
    sh = W.make_shower(n, seed=3, xmax=500.0, zenith_deg=20.0, azimuth_deg=15.0, beta="R")
    seg, geom, _ = cphot.upload(sh.seg, np.array([[*sh.core, *sh.axis]]), None)
    return cphot.make_segments(seg, geom)


def _run(S, det, side, n_t=0):
    bins = torch.zeros(side * side, dtype=torch.int64, device="cuda")
    times = torch.zeros(side * side * (n_t + 1), dtype=torch.int32, device="cuda") if n_t else None
    cnt = torch.zeros(cphot.NCOUNTERS, dtype=torch.int64, device="cuda")
    cphot.propagate(S, det, bins, times, cnt)
    return [t for t in (bins, times, cnt) if t is not None]


# the largest square arrays of a block that may take 64 KB beside the tables it held when
# they were set: 12,944, 12,044, 11,660 and 7,408 spheres at 128, fewer above
@pytest.mark.parametrize("transport,block,side",
                         [("straight", 128, 113), ("layered", 128, 109), ("table", 128, 107), ("surrogate", 128, 86),
                          ("straight", 128, 100), ("straight", 256, 98), ("layered", 256, 93), ("table", 256, 92),
                          ("surrogate", 256, 70), ("straight", 512, 54), ("layered", 512, 40), ("surrogate", 512, 40)])
def test_arrays_that_fit_are_held(transport, block, side):
    """Demanded (lds_hist 1) and by choice, with and without arrival times: the counts of
    device atomics alone."""
    S = _segments(4000)
    for n_t in (0, 5):
        ref = _run(S, _detector(transport, side, n_t, block_size=128, lds_hist=0), side, n_t)
        assert int(ref[-1][7]) > 100
        for lds in (1, -1):
            got = _run(S, _detector(transport, side, n_t, block_size=block, lds_hist=lds), side, n_t)
            assert all(torch.equal(a, b) for a, b in zip(got, ref)), (n_t, lds)
