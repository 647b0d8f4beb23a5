"""Training sets over block edges, and shells thick enough for the general walk."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")

BOX = {"planar": (W.SURROGATE_LO, W.SURROGATE_HI), "curved": (W.SURROGATE_CURVED_LO, W.SURROGATE_CURVED_HI)}


@pytest.mark.parametrize("geometry", ["planar", "curved"])
@pytest.mark.parametrize("n,first", [(1, 0), (63, 5), (257, 0), (511, 1), (512, 0), (513, 7), (1025, 600)])
def test_samples_do_not_depend_on_their_block(geometry, n, first):
    """A sample is a function of its index alone: the same bits in a set of any size, from
    any first index, wherever the sort by start layer puts it."""
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    sur = cphot.Surrogate(*BOX[geometry], geometry=geometry)
    X, Y = sur.make_training_set(atm, n, seed=31, first=first)
    Xa, Ya = sur.make_training_set(atm, 2000, seed=31)
    assert torch.equal(X, Xa[first:first + n])
    assert torch.equal(Y, Ya[first:first + n])


@pytest.mark.parametrize("n_layers,cos_lo", [(2, 0.2), (4, 0.2), (128, 0.5), (128, 1.0)])
def test_thick_and_thin_shells_match_oracle(n_layers, cos_lo):
    """Chords of up to 250 km in one shell leave the arc sine's series; straight down the
    central angle is zero. Bounds: FP32 layer data and outputs are 6e-8 relative each, the
    path integrals' sums of one sign; 1e-6 of the target covers them. Per metre of chord
    1e-9 (1e-10 of optical depth) stands for the outputs that vanish straight down."""
    desc = dict(cases.ATMO_LAYERED, n_layers=n_layers)
    lo, hi = list(W.SURROGATE_CURVED_LO), list(W.SURROGATE_CURVED_HI)
    lo[0], hi[0] = 15000.0, 50000.0
    lo[1], hi[1] = cos_lo, 1.0
    desc["h_top"] = 50000.0
    if cos_lo == 1.0:
        lo[1], hi[1] = 0.9999999, 1.0
    atm, oatm = cphot.Atmosphere(**desc), O.Atmosphere(**desc)
    sur = cphot.Surrogate(lo, hi, geometry="curved")
    X, Y = sur.make_training_set(atm, 3000, seed=5)
    X, Y = X.cpu().numpy().astype(np.float64), Y.cpu().numpy().astype(np.float64)
    Yo = O.surrogate_targets(oatm, X, "curved")
    assert np.all(np.isfinite(Y))
    for o, atol in enumerate([1e-9, 1e-12, 1e-9, 1e-10]):
        assert np.all(np.abs(Y[:, o] - Yo[:, o]) <= 1e-6 * np.abs(Yo[:, o]) + atol), o
