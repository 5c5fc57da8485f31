"""The tile kernels' branches that small batches do not reach (those go to the
short kernels): fillers behind the sequences under test take a batch past each
line, and every test states which side it is on from the sizes and the number
of compute units."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2605_13433_amd import hstu, inputs
from tests.gpu_util import TOL, check, rows_of, say, to_dev
from tests.test_gpu_parity import far_timestamps

pytestmark = pytest.mark.gpu

# odd and even tile counts, one-tile and empty sequences, a 1-row last tile
LENGTHS = [256, 320, 64, 65, 1, 767, 0, 639]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def items(w):
    return hstu.max_entries(w.B, w.N, w.T) * w.H


def workload(filler, far=False, **kw):
    w = inputs.make_workload(LENGTHS + filler, N=768, **kw)
    if far:
        w.timestamps = far_timestamps(LENGTHS + filler, seed=51)
    return w


def run(w, alpha=1.0, backward=False):
    q, k, v, u, off = (to_dev(x) for x in (w.q, w.k, w.v, w.u, w.seq_offsets))
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets, backward=backward, alpha=alpha)
    f = plan.forward(q, k, v, u, off)
    out = dict(o=f.o, y=f.y)
    if backward:
        g = plan.backward(q, k, v, u, off, to_dev(w.dy))
        out.update(dq=g.dq, dk=g.dk, dv=g.dv, du=g.du, d_pos=g.d_pos_w, d_time=g.d_time_w)
    torch.cuda.synchronize()
    return {n: None if t is None else t.detach().to("cpu", torch.float64).numpy()
            for n, t in out.items()}


def compare(w, got, alpha, tables=False):
    """The sequences under test (and the last filler) against the oracle; the
    tables on the whole batch."""
    seqs = list(range(len(LENGTHS))) + [w.B - 1]
    sub, rows = inputs.subset(w, seqs), rows_of(w, seqs)
    ref = oracle.fwd_workload(sub, alpha=alpha)
    if "dq" in got:
        ref = dict(ref, **oracle.bwd_workload(sub, alpha=alpha))
    for n in ("o", "y", "dq", "dk", "dv", "du"):
        if n in got:
            check(n, got[n][rows], ref[n].reshape(got[n][rows].shape), TOL[w.dtype])
    if tables:
        full = oracle.bwd_workload(w, alpha=alpha)
        for n in ("d_pos", "d_time"):
            if got[n] is not None:
                check(n, got[n], full[n], TOL[w.dtype])


# all heads' time tables staged once (H = 4) and one head's an item (H = 8)
@pytest.mark.parametrize("H", [4, 8])
@pytest.mark.parametrize("pos,time,far", [(True, True, False), (True, True, True),
                                          (False, True, False), (False, True, True),
                                          (True, False, False), (False, False, False)])
def test_two_tile_forward(H, pos, time, far):
    say(f"two-tile forward H={H} pos={pos} time={time} far={far}")
    w = workload([700] * 50, far, H=H, d=64, pos=pos, time=time, seed=970 + H)
    # more items than any direct call takes, and long enough on average
    assert items(w) > 8 * cus() and w.T >= 256 * w.B
    for alpha in (1.0, -1.3):
        compare(w, run(w, alpha), alpha)


@pytest.mark.parametrize("d,H", [(64, 4), (64, 8), (128, 2)])
@pytest.mark.parametrize("pos,far", [(True, False), (True, True), (False, True)])
def test_one_tile_forward(d, H, pos, far):
    say(f"one-tile forward H={H} d={d} pos={pos} far={far}")
    w = workload([60] * 600, far, H=H, d=d, pos=pos, seed=980 + H)
    assert w.B > 128 and items(w) > 4 * cus() and w.T < 256 * w.B
    for alpha in (1.0, -1.3):
        compare(w, run(w, alpha), alpha)


# One launch over both item kinds, and two (see test_gpu_parity.py for the line).
@pytest.mark.parametrize("launches", [1, 2])
@pytest.mark.parametrize("d,H,nb,alpha", [(64, 2, 128, 1.0), (64, 4, 32, -1.3), (64, 8, 128, 0.7),
                                          (64, 2, 1, 1.0), (128, 2, 128, -1.3),
                                          (128, 4, 32, 1.0), (128, 1, 256, 0.7)])
def test_exact_time_backward(d, H, nb, alpha, launches):
    """Timestamps outside the float-exponent index in both launches of the
    tile kernels' backward, with every size of the d_time histogram."""
    say(f"exact time backward d={d} H={H} num_buckets={nb} alpha={alpha} launches={launches}")
    w = workload([60] * ((360 if launches == 1 else 16 * cus()) // H), True, H=H, d=d,
                 num_buckets=nb, seed=990 + d + H)
    assert 4 * items(w) > 2 * cus()                       # past the short kernels
    assert items(w) < 4 * cus() if launches == 1 else items(w) >= 16 * cus()
    compare(w, run(w, alpha, backward=True), alpha, tables=True)


@pytest.mark.parametrize("pos,time", [(True, True), (True, False), (False, True)])
def test_scale_backward_d128(pos, time):
    """A negative scale on the d = 128 tile kernels, ordinary timestamps."""
    w = workload([60] * 90, False, H=2, d=128, pos=pos, time=time, seed=1001)
    assert 4 * items(w) > cus() and items(w) < 4 * cus()
    say(f"negative scale d=128 pos={pos} time={time}")
    compare(w, run(w, -0.6, backward=True), -0.6, tables=True)
