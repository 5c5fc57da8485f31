"""The fp32 attention kernels at the edges of their 32-row items and of the
four waves' shares of the streamed side, against the float64 oracle at the
fp32 bound; infinities and NaNs reach only the rows whose causal pairs hold
them."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_2605_13433_amd import hstu, inputs
from tests.gpu_util import TOL, check, run_gpu, say, to_dev

pytestmark = pytest.mark.gpu

# one row, either side of a 32-row item, of a 64-row entry, and of four
# waves' 32-row tiles; a fifth tile
LENGTHS = [1, 31, 32, 33, 0, 63, 64, 65, 95, 127, 128, 129, 161, 257]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("pos,time,nb", [(True, True, 128), (False, True, 3000),
                                         (True, False, 128), (False, False, 128)])
def test_edges(d, pos, time, nb):
    say(f"fp32 edges d={d} pos={pos} time={time} num_buckets={nb}")
    w = inputs.make_workload(LENGTHS, H=2, d=d, N=257, dtype=torch.float32, pos=pos, time=time,
                             num_buckets=nb, seed=900 + d)
    got = run_gpu(w)
    ref = dict(oracle.fwd_workload(w), **oracle.bwd_workload(w))
    for n in ("o", "y", "dq", "dk", "dv", "du"):
        check(n, got[n], ref[n], TOL[w.dtype])
    if pos:
        check("d_pos", got["d_pos"], ref["d_pos"], TOL[w.dtype])
    if time:
        check("d_time", got["d_time"], ref["d_time"], TOL[w.dtype])


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("N", [128, 129])
def test_many_short_sequences(d, N):
    """Either side of the line (max_len 128) where work-groups of two waves
    take over from four, with more items than run at once."""
    rng = np.random.default_rng(930 + d)
    lengths = [1, 32, 33, 64, 97, 127, 128] + [int(x) for x in rng.integers(0, 129, size=70)]
    w = inputs.make_workload(lengths, H=4, d=d, N=N, dtype=torch.float32, seed=930 + d)
    got = run_gpu(w)
    ref = dict(oracle.fwd_workload(w), **oracle.bwd_workload(w))
    for n in ("o", "y", "dq", "dk", "dv", "du", "d_pos", "d_time"):
        check(n, got[n], ref[n], TOL[w.dtype])


@pytest.mark.parametrize("d", [32, 64, 128])
def test_nonfinite_rows_stay_causal(d):
    """An infinite v (or k) row at position p leaves o (and dq) of the rows
    before p as they are, and an infinite dy row the dk and dv of the keys
    after it, bit for bit."""
    L, p = 150, 75
    w = inputs.make_workload([L], H=1, d=d, N=L, dtype=torch.float32, seed=910 + d)
    q, k, v, u = (to_dev(x) for x in (w.q, w.k, w.v, w.u))
    off, dy = to_dev(w.seq_offsets), to_dev(w.dy)
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets)

    def passes(k, v, dy):
        f = plan.forward(q, k, v, u, off)
        o, mean = f.o.clone(), f.ln_mean.clone()
        g = plan.backward(q, k, v, u, off, dy)
        torch.cuda.synchronize()
        return o, mean, g.dq.clone(), g.dk.clone(), g.dv.clone()

    base = passes(k, v, dy)
    for bad in (float("inf"), float("nan")):
        kb, vb, yb = k.clone(), v.clone(), dy.clone()
        vb[p, 0, 3] = bad
        o = passes(k, vb, dy)[0]
        assert torch.equal(o[:p], base[0][:p]), "o before the row"
        assert not torch.isfinite(o[p:, 0, 3]).any()
        kb[p, 0, 5] = bad
        dq = passes(kb, v, dy)[2]
        assert torch.equal(dq[:p], base[2][:p]), "dq before the row"
        yb[p] = bad
        _, _, _, dk, dv = passes(k, v, yb)
        assert torch.equal(dk[p + 1:], base[3][p + 1:]), "dk after the row"
        assert torch.equal(dv[p + 1:], base[4][p + 1:]), "dv after the row"
        assert not np.isfinite(dv[:p + 1].cpu().numpy()).any()


@pytest.mark.parametrize("d", [32, 64, 128])
def test_cancelling_biases(d):
    """Position and time biases of 1000 that cancel to about one: the score keeps
    the precision of their sum (rounded at 1000 on the way it is off by 3e-5,
    three times the bound)."""
    w = inputs.make_workload([97, 1, 130, 64], H=2, d=d, N=130, dtype=torch.float32, seed=940 + d)
    w.pos_w += 1000.0
    w.time_w -= 1000.0
    got = run_gpu(w)
    ref = dict(oracle.fwd_workload(w), **oracle.bwd_workload(w))
    for n in ("o", "y", "dq", "dk", "dv", "du", "d_pos", "d_time"):
        check(n, got[n], ref[n], TOL[w.dtype])
