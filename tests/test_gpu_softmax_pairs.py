"""GPU: fp32 attention softmax of 2 Mi scores and more with rows of whole 128-byte lines, whose packs lie in lane pairs: each sentence of such a call
against the call of this sentence alone, which is too small for that form and is checked against the CPU oracle elsewhere, bit for bit: both
add in the order of a row's packs."""
import numpy as np
import pytest
import torch

import paper_2110_05722_amd as L
from tests._util import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Lk", [64, 96, 128, 160, 288, 544, 1056, 1568, 2048, 2080, 4128, 8224, 16384])
def test_large_calls_and_their_sentences(Lk, causal):
    say(f"[softmax pairs] keys {Lk} causal {causal}")
    d = dev()
    N, Lq, scale = 2, 40 if Lk < 2048 else 9, 0.7
    B = (1 << 21) // (N * Lq * Lk) + 2
    g = torch.Generator(device=d).manual_seed(Lk)
    x, dy = (torch.randn(B, N, Lq, Lk, generator=g, device=d) * 2 for _ in range(2))
    kl = torch.randint(0, Lk + 1, (B,), generator=g, device=d, dtype=torch.int32)
    ql = torch.randint(0, Lq + 1, (B,), generator=g, device=d, dtype=torch.int32)
    kl[0], ql[0], kl[-1], ql[-1], kl[B // 2] = Lk - 3, Lq, 5, Lq - 1, Lk
    out = torch.arange(Lk, device=d)[None, None, None, :] >= kl[:, None, None, None]
    x, dy = x.masked_fill(out, float("nan")), dy.masked_fill(out, float("inf"))        # what lies behind the keys never counts
    x[-1, 0, 0, 1], dy[0, 1, 2, 3] = float("nan"), float("inf")                        # rows that are spoilt inside the mask
    for p in (0.0, 0.2):
        for lens in ((None, None), (kl, None), (kl, ql)):
            if lens[0] is None:
                xs, dys = torch.nan_to_num(x), torch.nan_to_num(dy, posinf=1.0)
            else:
                xs, dys = x, dy
            y, yd = L.lsq_softmax_varlen_fwd(xs, *lens, causal, scale, p, 3, 5)
            dx = L.lsq_softmax_varlen_bwd(dys, y, *lens, causal, scale, p, 3, 5)
            for b in ((0,) if p else (0, B // 2, B - 1)):                              # (the draws count from the tensor's start)
                one = [None if v is None else v[b:b + 1].contiguous() for v in lens]
                y1, yd1 = L.lsq_softmax_varlen_fwd(xs[b:b + 1].contiguous(), *one, causal, scale, p, 3, 5)
                yb = y[b:b + 1].contiguous()
                assert torch.equal(yb.view(torch.int32), y1.view(torch.int32))
                if p:
                    assert torch.equal(yd[b:b + 1].contiguous().view(torch.int32), yd1.view(torch.int32))
                dx1 = L.lsq_softmax_varlen_bwd(dys[b:b + 1].contiguous(), yb, *one, causal, scale, p, 3, 5)
                assert torch.equal(dx[b:b + 1].contiguous().view(torch.int32), dx1.view(torch.int32))
            xi, di = xs.clone(), dys.clone()                                           # in place
            if not p:
                assert torch.equal(torch.nan_to_num(L.lsq_softmax_varlen_fwd(xi, *lens, causal, scale, p, 3, 5, y=xi)[0]), torch.nan_to_num(y))
            assert torch.equal(torch.nan_to_num(L.lsq_softmax_varlen_bwd(di, y, *lens, causal, scale, p, 3, 5, dx=di)), torch.nan_to_num(dx))


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("Lk,lanes", [(64, 8), (128, 8), (256, 16), (512, 32), (1024, 64)])
def test_order_of_a_rows_sum(Lk, lanes, large):
    """Backward with y = 1 and scale 1: dx = dy - sum(dy).  The sum in float32, in the documented order: a lane adds its packs (lanes apart) element by
    element, then the lanes meet by ascending bits of the pack's index."""
    say(f"[softmax pairs] order of the sum, {Lk} keys, {'large' if large else 'small'} call")
    d = dev()
    rows = (1 << 21) // Lk + 3 if large else 37
    dy = torch.randn((1, 1, rows, Lk), generator=torch.Generator().manual_seed(Lk)) * 100
    dx = L.lsq_softmax_bwd(dy.to(d), torch.ones_like(dy, device=d), None, False, 1.0, 0.0, 1, 1).cpu().numpy().reshape(rows, Lk)
    v = dy.numpy().reshape(rows, -1, lanes, 8)
    acc = np.zeros((rows, lanes), np.float32)
    for k in range(v.shape[1]):
        for j in range(8):
            acc += v[:, k, :, j]
    while acc.shape[1] > 1:
        acc = acc[:, 0::2] + acc[:, 1::2]
    assert np.array_equal(dx, dy.numpy().reshape(rows, Lk) - acc)
