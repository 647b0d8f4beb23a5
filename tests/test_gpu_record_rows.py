"""List mode: rows in buffers that begin between 16-byte boundaries, with gaps between the
segments, and of capacities that end inside a round of records."""
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")

ROW = cphot.RECORD_BYTES


@pytest.mark.parametrize("block", [0, 128, 512])
@pytest.mark.parametrize("transport,zenith", [("straight", 0.0), ("layered", 30.0), ("curved", 70.0)])
def test_rows_land_where_they_belong(transport, zenith, block):
    """The same bytes in a packed buffer and in one that begins 8 bytes past a boundary,
    with gaps between the segments and an end inside the records; nothing else is written."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    n = 200
    seg, offs, geom = W.concat_showers([W.make_shower(n, seed=61, zenith_deg=zenith, beta="R", dedx=(0.1, 2.0))])
    S = cphot.make_segments(*cphot.upload(seg, geom, offs))
    det = cphot.make_detector(atm, transport=transport, spectrum="frank_tamm", seed=4, emission="both", nx=80,
                              ny=60, cell=20.0, block_size=block)
    counts = torch.empty(n, dtype=torch.int32, device="cuda")
    cphot.segment_counts(S, det, counts)
    total = int(counts.sum())
    assert total > 64 * n // 8
    first = torch.cumsum(counts, 0, dtype=torch.int64) - counts
    packed = torch.zeros(total * ROW, dtype=torch.uint8, device="cuda")
    cphot.trace_records(S, det, first, packed)
    rows = packed.view(total, ROW)

    own = torch.repeat_interleave(torch.arange(n, device="cuda"), counts.long())
    gaps = torch.arange(n, device="cuda") % 5 + 1
    at = first + torch.cumsum(gaps, 0)
    place = at[own] + torch.arange(total, device="cuda") - first[own]
    for cap in (int(place[-1]) + 3, int(place[total // 2]) + 1, int(place[70]), 1):
        buf = torch.full((8 + (cap + 70) * ROW,), 0xA5, dtype=torch.uint8, device="cuda")
        cphot.trace_records(S, det, at, buf[8:8 + cap * ROW])
        want = torch.full((cap + 70, ROW), 0xA5, dtype=torch.uint8, device="cuda")
        inside = place < cap
        want[place[inside]] = rows[inside]
        assert torch.equal(buf[8:].view(cap + 70, ROW), want), cap
        assert bool((buf[:8] == 0xA5).all())
