"""A sequence's outputs do not depend on the batch around it, bit for bit: the
same sequences in a batch small enough for the short kernels (32-row items)
and in batches past that line, where the tile kernels' one-tile, direct and
two-tile items take them.  Ragged lengths at the edges of the 32-row items,
of the waves' shares and of the 64-row tiles."""
import pytest
import torch

from paper_2605_13433_amd import hstu, inputs
from tests.gpu_util import say, to_dev
from tests.test_gpu_parity import far_timestamps

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 32, 33, 0, 63, 64, 65, 96, 127, 128, 129, 161, 200]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def forward_is_short(w):
    """The forward's line: every 32-row item's work-group runs at once, three
    on a compute unit at d = 64 and one at d = 128."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return 2 * hstu.max_entries(w.B, w.N, w.T) * w.H <= (3 if w.d == 64 else 1) * cus


def forward(w, alpha=1.0):
    q, k, v, u, off = (to_dev(x) for x in (w.q, w.k, w.v, w.u, w.seq_offsets))
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets, backward=False, alpha=alpha)
    f = plan.forward(q, k, v, u, off)
    torch.cuda.synchronize()
    return dict(o=f.o, y=f.y, mean=f.ln_mean, rstd=f.ln_rstd)


def batches(lengths, filler, far, **kw):
    """The sequences of `lengths` alone, and with `filler` behind them."""
    w = inputs.make_workload(lengths + filler, **kw)
    if far:
        w.timestamps = far_timestamps(lengths + filler, seed=31)
    return inputs.subset(w, list(range(len(lengths)))), w


# fillers: past the short kernels alone; past the direct forward's 128
# sequences too; long enough for the two-tile items at d = 64 (mean length 256
# and more)
@pytest.mark.parametrize("filler", [[90] * 100, [40] * 420, [650] * 40],
                         ids=["direct", "many", "long"])
@pytest.mark.parametrize("pos,time,far", [(True, True, False), (True, True, True),
                                          (True, False, False), (False, True, False),
                                          (False, True, True), (False, False, False)])
@pytest.mark.parametrize("d", [64, 128])
def test_forward_bits(d, pos, time, far, filler):
    say(f"batch bits forward d={d} pos={pos} time={time} far={far} filler={len(filler)}")
    for alpha in (1.0, 0.3):
        small, large = batches(LENGTHS, filler, far, H=2, d=d, N=700, pos=pos, time=time,
                               seed=600 + d)
        assert forward_is_short(small) and not forward_is_short(large)
        a, b = forward(small, alpha), forward(large, alpha)
        for n in a:
            assert torch.equal(a[n], b[n][:small.T]), n


@pytest.mark.parametrize("d,B", [(64, 1), (128, 1), (64, 3)])
def test_forward_bits_long(d, B):
    """Many tiles a wave, the last step ragged."""
    small, large = batches([1650, 700, 31][:B], [650] * 40, False, H=2, d=d, N=1700, seed=610 + d)
    assert forward_is_short(small) and not forward_is_short(large)
    a, b = forward(small), forward(large)
    for n in a:
        assert torch.equal(a[n], b[n][:small.T]), n
