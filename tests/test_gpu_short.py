"""The kernels for short batches (32-row items, four independent waves)
against the oracle, beside the tile kernels on the same sequences: three
hundred and more one-token sequences behind them take the batch past the line
between the two.  Ragged lengths at the edges of the 32-row items and of the
waves' shares, each bias combination, the score scale, deterministic tables,
timestamps that leave the float-exponent index, infinities before and after
a row."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2605_13433_amd import hstu, inputs
from tests.gpu_util import TOL, check, say, to_dev
from tests.test_gpu_parity import far_timestamps

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 32, 33, 0, 63, 64, 65, 96, 127, 128, 129, 161, 200]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


def gpu(w, alpha=1.0, det=False):
    q, k, v, u, off = (to_dev(x) for x in (w.q, w.k, w.v, w.u, w.seq_offsets))
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets, alpha=alpha, deterministic=det)
    f = plan.forward(q, k, v, u, off)
    g = plan.backward(q, k, v, u, off, to_dev(w.dy))
    torch.cuda.synchronize()
    out = dict(o=f.o, y=f.y, dq=g.dq, dk=g.dk, dv=g.dv, du=g.du, d_pos=g.d_pos_w,
               d_time=g.d_time_w)
    return {n: t.detach().cpu() for n, t in out.items() if t is not None}


def against_oracle(w, got, alpha=1.0):
    ref = dict(oracle.fwd_workload(w, alpha=alpha), **oracle.bwd_workload(w, alpha=alpha))
    for n, t in got.items():
        a = t.to(torch.float64).numpy()
        check(n, a, ref[n].reshape(a.shape), TOL[w.dtype])


@pytest.mark.parametrize("filler", [0, 330])
@pytest.mark.parametrize("pos,time", [(True, True), (True, False), (False, True), (False, False)])
@pytest.mark.parametrize("d", [64, 128])
def test_edges(d, pos, time, filler):
    say(f"short edges d={d} pos={pos} time={time} filler={filler}")
    w = inputs.make_workload(LENGTHS + [1] * filler, H=2, d=d, N=200, pos=pos, time=time,
                             seed=810 + d)
    against_oracle(w, gpu(w))


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("H,nb", [(1, 256), (1, 512), (2, 128), (2, 129), (4, 64), (4, 128)])
@pytest.mark.parametrize("d", [64, 128])
def test_tile_time_histograms(d, H, nb, det):
    """The tile kernels' d_time histogram on both sides of its lines: all heads'
    to the work-group's end or the item's head's, one to eight counters.
    (The batch is filled past the short kernels with 40-token sequences: with
    one head the LayerNorm makes a one-token sequence's dO orthogonal to its o,
    a multiple of v, so its dS = <dO, v> is a cancellation; 700 of them sum |dS|
    to 20 times the largest table entry, and rounding o and dO to bf16 alone
    moves the diagonal's sum by 1% of it at d=128, half the tolerance.)"""
    w = inputs.make_workload(LENGTHS + [40] * 300, H=H, d=d, N=200, num_buckets=nb, seed=850 + d)
    against_oracle(w, gpu(w, det=det))


@pytest.mark.parametrize("d,N,nb", [(64, 200, 32), (128, 200, 2048), (64, 3, 1)])
def test_scale_deterministic_far(d, N, nb):
    """A score scale, fixed-point tables that repeat bit for bit, bucket
    counts with one and with eight histogram copies, far timestamps, and a
    table narrower than a tile."""
    lengths = [min(L, N) for L in LENGTHS]
    w = inputs.make_workload(lengths, H=2, d=d, N=N, num_buckets=nb, seed=820 + d)
    w.timestamps = far_timestamps(lengths, seed=821)
    for alpha in (0.125, -1.3):
        say(f"short alpha={alpha} deterministic d={d} num_buckets={nb}")
        a, b = gpu(w, alpha, det=True), gpu(w, alpha, det=True)
        for n in a:
            assert torch.equal(a[n], b[n]), n
        against_oracle(w, a, alpha)


@pytest.mark.parametrize("H,B", [(1, 129), (1, 250), (64, 2)])
def test_lists_and_heads(H, B):
    """More sequences than a call finds without the scheduler; every head."""
    lengths = [1 + (b * 7) % 40 for b in range(B)]
    w = inputs.make_workload(lengths, H=H, d=64, N=64, num_buckets=32, seed=830)
    against_oracle(w, gpu(w))


@pytest.mark.parametrize("d", [64, 128])
def test_long_single_sequence(d):
    """Many tiles per wave, the last share ragged."""
    w = inputs.make_workload([1650], H=1, d=d, N=1700, seed=840 + d)
    against_oracle(w, gpu(w))


@pytest.mark.parametrize("d", [64, 128])
def test_nonfinite_stays_behind_its_tile(d):
    """An infinite v row leaves every row before its 32-row tile as it was,
    bit for bit, and an infinite dy row the keys after its tile."""
    L, p = 150, 70
    w = inputs.make_workload([L], H=1, d=d, N=L, seed=850 + d)
    base = gpu(w)
    vb = w.v.clone()
    w.v[p, 0, 3] = float("inf")
    bad = gpu(w)
    assert torch.equal(bad["o"][:64], base["o"][:64])
    assert not torch.isfinite(bad["o"][p:, 0, 3].float()).any()
    w.v = vb
    w.dy[p] = float("inf")
    bad = gpu(w)
    for n in ("dk", "dv"):
        assert torch.equal(bad[n][96:], base[n][96:]), n
    assert not np.isfinite(bad["dv"][:p + 1].float().numpy()).any()
