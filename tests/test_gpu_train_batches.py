"""The reduction of the training step at every kind of batch."""
import pytest

from paper_2405_04229_amd import workload as W
from tests import cases

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
cphot = pytest.importorskip("paper_2405_04229_amd.cphot")


def _surrogate(n):
    atm = cphot.Atmosphere(**cases.ATMO_LAYERED)
    sur = cphot.Surrogate(W.SURROGATE_LO, W.SURROGATE_HI, max_batch=8192, init_seed=3)
    X, Y = sur.make_training_set(atm, n, seed=12)
    sur.fit_normalization(Y)
    return sur, X, Y


@pytest.mark.parametrize("blocks", [7, 8, 9, 15, 16, 17, 48, 63, 96, 97, 127, 128])
def test_gradient_is_the_mean_of_its_blocks(blocks):
    """Around the numbers of loads in flight. Each block's residuals enter the backward pass
    rounded to bf16 (relative 2^-9, of either sign), scaled by another batch size in the two:
    the means agree to 2^-8. A partial left out or added twice is off by 1 / blocks of a
    gradient's size, more than that up to 128 blocks."""
    sur, X, Y = _surrogate(64 * blocks)
    g, loss = sur.gradient(X, Y)
    parts = [sur.gradient(X[64 * b:64 * b + 64].contiguous(), Y[64 * b:64 * b + 64].contiguous()) for b in range(blocks)]
    each = torch.stack([p[0] for p in parts]).double()
    assert float((g.double() - each.mean(0)).norm()) <= 2.0 ** -8 * float(each.norm()) / blocks ** 0.5
    assert float(loss) == pytest.approx(float(torch.stack([p[1] for p in parts]).double().mean()), rel=1e-5)


@pytest.mark.parametrize("blocks,more", [(63, 64), (56, 64), (127, 128)])
def test_a_smaller_batch_is_no_slower(blocks, more):
    """100 steps of a batch that is some blocks short of a multiple of 64 partials take no
    longer than the batch that is not (twice as long with the rest added load by load): within
    a tenth, two runs of one batch differing by 2 %."""
    times = []
    for k in (blocks, more):
        sur, X, Y = _surrogate(64 * more)
        best = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            sur.train(X, Y, batch=64 * k, steps=100, lr=1e-3)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[0] < 1.1 * times[1], times
