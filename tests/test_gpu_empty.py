"""Backward calls without tokens, down to one sequence and none: they succeed
and write every entry of the bias tables' gradients (and the layer's weight
gradients) as zero."""
import pytest
import torch

from paper_2605_13433_amd import hstu
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def tables(H, N, nb):
    return (torch.randn(H, 2 * N - 1, device="cuda"), torch.randn(H, nb, device="cuda"),
            torch.empty(0, dtype=torch.int64, device="cuda"))


def zero(*tensors):
    torch.cuda.synchronize()
    for t in tensors:
        assert torch.count_nonzero(t).item() == 0


@pytest.mark.parametrize("B", [0, 1, 2])
@pytest.mark.parametrize("d,dtype", [(64, BF), (128, BF), (32, F32)])
def test_attention(B, d, dtype):
    H, N, nb = 2, 70, 40
    say(f"backward of {B} sequences without tokens, d={d} {dtype}")
    pos, time, ts = tables(H, N, nb)
    off = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
    x = torch.empty(0, H, d, dtype=dtype, device="cuda")
    for det in (False, True):
        plan = hstu.Plan(x, off, N, pos, time, ts, nb, deterministic=det)
        plan.forward(x, x, x, x, off)
        plan.d_pos.fill_(7.0)
        plan.d_time.fill_(7.0)
        g = plan.backward(x, x, x, x, off, torch.empty(0, H * d, dtype=dtype, device="cuda"))
        zero(g.d_pos_w, g.d_time_w)


@pytest.mark.parametrize("B", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_layer(B, d):
    H, N, nb, D = 2, 70, 40, 64
    say(f"layer backward of {B} sequences without tokens, d={d}")
    pos, time, ts = tables(H, N, nb)
    off = torch.zeros(B + 1, dtype=torch.int64, device="cuda")
    x = torch.empty(0, D, dtype=BF, device="cuda")
    w1 = torch.randn(D, 4 * H * d, device="cuda").to(BF)
    w2 = torch.randn(H * d, D, device="cuda").to(BF)
    plan = hstu.LayerPlan(x, off, N, H, d, pos, time, ts, nb)
    plan.forward(x, w1, w2, off)
    for t in (plan.grad.dw1, plan.grad.dw2, plan.grad.d_pos_w, plan.grad.d_time_w):
        t.fill_(7.0)
    g = plan.backward(x, w1, w2, off, torch.empty(0, D, dtype=BF, device="cuda"))
    zero(g.dw1, g.dw2, g.d_pos_w, g.d_time_w)
