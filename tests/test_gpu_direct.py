"""Forward calls small enough to run every item at once find their items
without the scheduler; with the offsets check on (HSTU_VALIDATE=1) the same
call goes through the scheduler's lists.  Both must give the same bits: an
item's arithmetic does not depend on how it was found."""
import pytest
import torch

from oracle import oracle
from paper_2605_13433_amd import hstu, inputs
from tests.gpu_util import TOL, check, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


CASES = [
    # lengths, H, d, dtype: one entry; empty sequences around and between;
    # 63/64/65-row tails; the second 64 sequences of a wave; the last batch
    # size taken directly and the first that is not; few long ones
    ([1], 1, 64, torch.bfloat16),
    ([0, 0, 63, 0, 64, 65, 0, 129, 0], 2, 128, torch.bfloat16),
    ([(37 * b) % 90 for b in range(128)], 2, 64, torch.bfloat16),
    ([1 + b % 3 for b in range(129)], 2, 64, torch.bfloat16),
    ([700, 3, 513], 2, 64, torch.bfloat16),
    ([0, 33, 64, 0, 65, 1], 2, 32, torch.float32),
    ([(29 * b) % 70 for b in range(100)], 1, 64, torch.float32),
    # past the short kernels' line (2 items of 32 rows to an entry and head, three
    # work-groups a compute unit at d=64 and one at d=128), and still direct: the
    # tile kernels' one-tile items, beside one- and two-tile ones from the lists
    ([90] * 110, 2, 128, torch.bfloat16),
    ([130, 1, 0, 64] * 30, 3, 64, torch.bfloat16),
    ([700] * 20 + [3, 513], 2, 64, torch.bfloat16),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("noalloc", [False, True])
def test_direct_equals_lists(case, noalloc, monkeypatch):
    lengths, H, d, dtype = CASES[case]
    say(f"direct forward case {case}: {len(lengths)} sequences H={H} d={d} noalloc={noalloc}")
    w = inputs.make_workload(lengths, H=H, d=d, N=max(lengths) + 5, dtype=dtype, seed=700 + case)
    q, k, v, u, off = (to_dev(x) for x in (w.q, w.k, w.v, w.u, w.seq_offsets))
    plan = hstu.Plan(q, off, w.N, to_dev(w.pos_w), to_dev(w.time_w), to_dev(w.timestamps),
                     w.num_buckets, backward=False)

    def run(validate):
        monkeypatch.setenv("HSTU_VALIDATE", validate)
        for t in (plan.y, plan.o, plan.mean, plan.rstd):
            t.fill_(float("nan"))
        if noalloc:
            hstu.hstu_jagged_attn_fwd_noalloc(q, k, v, u, off, plan.B, w.N, H, d, plan.rab,
                                              plan.out)
            st = None
        else:
            plan.forward(q, k, v, u, off)
            st = plan.status()
        torch.cuda.synchronize()
        return [t.clone() for t in (plan.y, plan.o, plan.mean, plan.rstd)], st

    direct, st_direct = run("0")
    lists, st_lists = run("1")
    for a, b in zip(direct, lists):
        assert torch.equal(a, b)
    if not noalloc:
        assert st_direct == hstu.HSTU_SEQ_UNCHECKED and st_lists == 0
    ref = oracle.fwd_workload(w)
    check("o", direct[1].double().cpu().numpy(), ref["o"], TOL[dtype])
    check("y", direct[0].double().cpu().numpy().reshape(ref["y"].shape), ref["y"], TOL[dtype])
