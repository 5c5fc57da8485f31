"""A sequence's outputs do not depend on the batch around it, bit for bit: the
same sequences in a batch small enough for the short kernels (32-row items)
and in batches past that line, where the tile kernels' one-tile, direct and
two-tile items and both launches of the backward take them.  Ragged lengths at
the edges of the 32-row items, of the waves' shares and of the 64-row tiles.
(The one exception is in the tile kernels alone: at d = 64 the backward in two
launches rounds dQ of a sequence's first 64 rows otherwise than the one in one.)"""
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


def backward_is_short(w):
    """The backward's: two work-groups an item, two on a compute unit (one at
    d = 128)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return 4 * hstu.max_entries(w.B, w.N, w.T) * w.H <= (2 if w.d == 64 else 1) * cus


def run(w, alpha=1.0, backward=False):
    q, k, v, u, off = (to_dev(x) for x in (w.q, w.k, w.v, w.u, w.seq_offsets))
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets, backward=backward, alpha=alpha)
    f = plan.forward(q, k, v, u, off)
    out = dict(o=f.o, y=f.y, mean=f.ln_mean, rstd=f.ln_rstd)
    if backward:
        g = plan.backward(q, k, v, u, off, to_dev(w.dy))
        out.update(dq=g.dq, dk=g.dk, dv=g.dv, du=g.du)
    torch.cuda.synchronize()
    return out


def same(small, large, names, **kw):
    a, b = run(small, **kw), run(large, **kw)
    for n in names:
        assert torch.equal(a[n], b[n][:small.T]), n


FORWARD, BACKWARD = ("o", "y", "mean", "rstd"), ("dq", "dk", "dv", "du")


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
        same(small, large, FORWARD, alpha=alpha)


@pytest.mark.parametrize("d,B", [(64, 1), (128, 1), (64, 3)])
def test_forward_bits_long(d, B):
    """Many tiles a wave, the last step ragged."""
    small, large = batches([1650, 700, 31][:B], [650] * 40, False, H=2, d=d, N=1700, seed=610 + d)
    assert forward_is_short(small) and not forward_is_short(large)
    same(small, large, FORWARD)


def two_launches(w):
    """Past this many items (4 for each of at most 4 work-groups a compute
    unit) the tile kernels' backward is two launches; it is one below 4 for each
    of one work-group."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    items = hstu.max_entries(w.B, w.N, w.T) * w.H
    assert items >= 16 * cus or items < 4 * cus
    return items >= 16 * cus


@pytest.mark.parametrize("filler", [[100] * 60, [40] * 1500], ids=["one", "two"])
@pytest.mark.parametrize("pos,time,far", [(True, True, False), (True, True, True),
                                          (True, False, False), (False, True, False),
                                          (False, True, True), (False, False, False)])
@pytest.mark.parametrize("d", [64, 128])
def test_backward_bits(d, pos, time, far, filler):
    say(f"batch bits backward d={d} pos={pos} time={time} far={far} filler={len(filler)}")
    small, large = batches(LENGTHS[:-2] if d == 128 else LENGTHS, filler, far, H=2, d=d, N=700,
                           pos=pos, time=time, seed=620 + d)
    assert backward_is_short(small) and not backward_is_short(large)
    assert two_launches(large) == (len(filler) == 1500)
    names = BACKWARD[1:] if d == 64 and two_launches(large) else BACKWARD
    for alpha in (1.0, -0.7):
        same(small, large, names, alpha=alpha, backward=True)


@pytest.mark.parametrize("d,L", [(64, 1650), (128, 1650), (64, 1027)])
def test_backward_bits_long(d, L):
    small, large = batches([L], [100] * 60, False, H=2, d=d, N=1700, seed=630 + d)
    assert backward_is_short(small) and not backward_is_short(large)
    same(small, large, BACKWARD, backward=True)


def f32_waves(w, per):
    """Two where sequences have at most four 32-row tiles and the work-groups
    (`per` to a list entry and head) queue for the device, else four."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    resident = 1 if w.d == 128 else 3 if w.d == 32 and per == 2 else 2
    queue = per * hstu.max_entries(w.B, w.N, w.T) * w.H > resident * cus
    return 2 if w.N <= 128 and queue else 4


@pytest.mark.parametrize("pos,time", [(True, True), (False, False)])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_f32_bits(d, pos, time):
    """fp32: work-groups of four waves and of two."""
    say(f"batch bits fp32 d={d} pos={pos} time={time}")
    lengths = [1, 31, 32, 33, 0, 63, 64, 65, 95, 96, 97, 127, 128]
    small, large = batches(lengths, [70] * 300, False, H=2, d=d, N=128, dtype=torch.float32,
                           pos=pos, time=time, seed=640 + d)
    small = inputs.subset(small, [0, 1, 3, 4, 7, 10, 12])
    assert f32_waves(small, 4) == 4 and f32_waves(large, 2) == 2
    off = large.seq_offsets.tolist()
    rows = torch.cat([torch.arange(off[b], off[b + 1]) for b in (0, 1, 3, 4, 7, 10, 12)]).cuda()
    a, b = run(small, backward=True), run(large, backward=True)
    for n in FORWARD + BACKWARD:
        assert torch.equal(a[n], b[n][rows]), n
