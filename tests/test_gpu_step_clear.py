"""A step clears all its outputs and nothing beside them, wherever they begin."""
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("dtype,nx,ny,detector", [("int32", 9, 9, "grid"), ("int32", 101, 97, "grid"),
                                                  ("float64", 61, 3, "grid"), ("int64", 5, 5, "spheres")])
def test_replays_equal_one_propagation(dtype, nx, ny, detector, shift):
    """Outputs between 16-byte boundaries, of odd lengths, filled with ones before each of
    three replays: equal to one propagation into zeros; the words around them stay."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    seg, offs, geom = W.concat_showers([W.make_shower(300, seed=5, zenith_deg=20.0, beta="R")])
    S = cphot.make_segments(*cphot.upload(seg, geom, offs))
    kw = dict(nx=nx, ny=ny, cell=20.0) if detector == "grid" else dict(snx=nx, sny=ny, pitch=150.0, radius=30.0, n_t=31, dt=1.0)
    det = cphot.make_detector(atm, transport="layered", detector=detector, spectrum="frank_tamm", seed=3, **kw)
    cells, times = nx * ny, nx * ny * 32
    dt = getattr(torch, dtype)

    def buffers():
        b = torch.ones(cells + 8, dtype=dt, device="cuda")
        t = torch.ones(times + 8, dtype=torch.int32, device="cuda") if detector == "spheres" else None
        c = torch.ones(cphot.NCOUNTERS + 8, dtype=torch.int64, device="cuda")
        return [(x, x[shift:shift + n]) if x is not None else (None, None)
                for x, n in ((b, cells), (t, times), (c, cphot.NCOUNTERS))]

    ref = buffers()
    for _, v in ref:
        if v is not None:
            v.zero_()
    cphot.propagate(S, det, *[v for _, v in ref])
    got = buffers()
    step = cphot.Step(S, det, *[v for _, v in got])
    for _ in range(3):
        for _, v in got:
            if v is not None:
                v.fill_(1)
        step.launch()
        torch.cuda.synchronize()
        for (a, _), (b, _) in zip(ref, got):
            assert a is None or torch.equal(a, b)
    assert int(ref[2][1][3]) > 0
