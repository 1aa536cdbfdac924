"""GPU: calls on both sides of the size from which a streamed input is loaded past the caches (16 MiB a tensor): the first rows of a call above it are, bit for bit,
the call of these rows alone, which is below it and checked against the CPU oracle elsewhere.  fp32 covers the packs in lane pairs (row ends inside a group
of lanes, heads of 64, 128 and 80 columns) as well."""
import pytest
import torch

import paper_2110_05722_amd as L
from tests._util import dev, say

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
LIMIT = 16 << 20


def _rows(width, dt):
    """rows of a call above the limit, and of one below it"""
    at = LIMIT // (width * DT[dt].itemsize)
    return at + 9, max(1, at // 2 + 1)


@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("width", [1024, 1032, 1280, 4104])
def test_elementwise_rows(width, dt):
    say(f"[cached loads] rows of {width} {dt}")
    g = torch.Generator(device=dev()).manual_seed(width)
    big, small = _rows(width, dt)
    r = lambda *s: torch.randn(s, generator=g, device=dev()).to(DT[dt])  # noqa: E731
    x, res, dy, bias = r(big, width), r(big, width), r(big, width), r(width)
    for p in (0.0, 0.3):
        assert torch.equal(L.lsq_bias_dropout_residual_fwd(x, bias, res, p, 1, 2)[:small], L.lsq_bias_dropout_residual_fwd(x[:small], bias, res[:small], p, 1, 2))
        assert torch.equal(L.lsq_bias_dropout_residual_bwd(dy, p, 1, 2)[0][:small], L.lsq_bias_dropout_residual_bwd(dy[:small], p, 1, 2)[0])
        for act in ("relu", "gelu"):
            assert torch.equal(L.lsq_bias_act_dropout_fwd(x, bias, act, p, 1, 2)[:small], L.lsq_bias_act_dropout_fwd(x[:small], bias, act, p, 1, 2))
            assert torch.equal(L.lsq_bias_act_dropout_bwd(dy, x, bias, act, p, 1, 2)[0][:small], L.lsq_bias_act_dropout_bwd(dy[:small], x[:small], bias, act, p, 1, 2)[0])


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("heads,head_dim,parts", [(8, 64, 3), (5, 128, 1), (7, 80, 2), (9, 64, 1)])
def test_heads(heads, head_dim, parts, dt):
    say(f"[cached loads] heads {heads} x {head_dim} x {parts} {dt}")
    g = torch.Generator(device=dev()).manual_seed(heads)
    ln, hidden = 33, heads * head_dim
    big = LIMIT // (ln * hidden * DT[dt].itemsize) + 2
    small = max(1, big // (2 * parts))
    r = lambda *s: torch.randn(s, generator=g, device=dev()).to(DT[dt])  # noqa: E731
    x, bias = r(big * ln, parts * hidden), r(parts * hidden)
    for b in (None, bias):
        for whole, part in zip(L.lsq_split_heads_fwd(x, b, big, ln, heads, head_dim, parts), L.lsq_split_heads_fwd(x[:small * ln], b, small, ln, heads, head_dim, parts)):
            assert whole is part is None or torch.equal(whole[:small], part)
    d = [r(big, heads, ln, head_dim) for _ in range(parts)]
    din, dbias = L.lsq_split_heads_bwd(d, big, ln, heads, head_dim)
    assert torch.equal(din[:small * ln], L.lsq_split_heads_bwd([t[:small].contiguous() for t in d], small, ln, heads, head_dim)[0])
    ref = din.double().sum(0)                  # fp32 sums of `rows` normal values: well within 1e-5 of their 2-norm
    assert (dbias.double() - ref).norm() <= 1e-5 * (din.shape[0] ** 0.5) * ref.shape[0] ** 0.5
    assert torch.equal(L.lsq_merge_heads_fwd(d[0])[:small * ln], L.lsq_merge_heads_fwd(d[0][:small].contiguous()))


@pytest.mark.parametrize("dt", ["f16", "f32"])
def test_padding(dt):
    say(f"[cached loads] padding {dt}")
    g = torch.Generator(device=dev()).manual_seed(3)
    ln, hidden = 40, 520
    big = LIMIT // (ln * hidden * DT[dt].itemsize) + 3
    x = torch.randn((big, ln, hidden), generator=g, device=dev()).to(DT[dt])
    lens = torch.full((big,), ln, dtype=torch.int32, device=dev())
    lens[1::3] = 17
    off = L.lsq_pad_offsets(lens, big, ln)
    keep = torch.arange(ln, device=dev())[None, :] < lens[:, None]
    packed = L.lsq_pad_remove(x, off, int(lens.sum()))
    assert torch.equal(packed, x[keep])
    full = torch.full((big,), ln, dtype=torch.int32, device=dev())
    foff = L.lsq_pad_offsets(full, big, ln)
    assert torch.equal(L.lsq_pad_restore(x.reshape(big * ln, hidden), foff, big, ln).reshape(x.shape), x)      # packed rows above the limit
    back = L.lsq_pad_restore(packed, off, big, ln).reshape(x.shape)
    assert torch.equal(back, torch.where(keep[..., None], x, torch.zeros_like(x)))
