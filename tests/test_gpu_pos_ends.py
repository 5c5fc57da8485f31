"""The position table's ends: sequences of max_len tokens reach its first entry
with their last query and first key, and the rows of a tile past them lie before
it; with a max_len of a few tokens four neighbouring entries end past it.  The
first entries are large, so that a pair that read another bias shows."""
import pytest
import torch

from oracle import oracle
from paper_2605_13433_amd import inputs
from tests.gpu_util import TOL, check, run_gpu, say

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 4, 5, 7, 31, 33, 34, 35, 66, 127, 130, 161, 162, 163, 501, 502, 503]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


# the short kernels' batches, the tile kernels', and fp32
@pytest.mark.parametrize("d,dtype,filler", [(64, torch.bfloat16, 0), (128, torch.bfloat16, 0),
                                            (64, torch.bfloat16, 400), (128, torch.bfloat16, 400),
                                            (32, torch.float32, 0), (64, torch.float32, 0),
                                            (128, torch.float32, 0)])
@pytest.mark.parametrize("time", [False, True])
def test_table_ends(d, dtype, filler, time):
    """o and dv, which are sums of the pairs' activations (dS hangs on <dO, v>,
    which the LayerNorm makes a cancellation where one bias outweighs the rest);
    the query-streaming and key-streaming items read every bias for one of them."""
    for N in SIZES:
        w = inputs.make_workload([N, max(N - 1, 1), N] + [min(N, 30)] * filler, H=2, d=d, N=N,
                                 dtype=dtype, time=time, seed=960 + N)
        w.pos_w *= 10.0
        w.pos_w[:, :4] += 30.0
        say(f"table ends N={N} d={d} {dtype} time={time} filler={filler}")
        got = run_gpu(w)
        ref = dict(oracle.fwd_workload(w), **oracle.bwd_workload(w))
        for n in ("o", "dv"):
            check(n, got[n][:N], ref[n][:N], TOL[dtype])
