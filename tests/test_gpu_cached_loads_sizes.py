"""GPU: the first and last rows of calls on both sides of the sizes between which a streamed input is loaded through the caches (2 and 16 MiB a tensor) and from which fp32
packs go in lane pairs (2 or 4 MiB). The first rows of a call above one are, bit for bit, the call of these rows alone, which is below it and checked against the CPU oracle elsewhere;
without dropout its last rows, a partial trip, are the call of those rows alone, and with dropout the result without, under the oracle's mask. Column sums against the
stored gradients in 64 bits. fp32 covers the packs in lane pairs (row ends inside a group of lanes, heads of 64, 128 and 80 columns) as well."""
import pytest
import torch

import oracle
import paper_2110_05722_amd as L
from tests._util import dev, say

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
LIMITS = [2 << 20, 4 << 20, 16 << 20]


def _rows(width, dt, limit):
    """rows of a call above the limit, and of one below it"""
    at = limit // (width * DT[dt].itemsize)
    return at + 9, max(1, at // 2 + 1)


@pytest.mark.parametrize("limit", LIMITS)
@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("width", [1024, 1032, 1280, 4104])
def test_elementwise_rows(width, dt, limit):
    say(f"[cached loads] rows of {width} {dt} about {limit}")
    g = torch.Generator(device=dev()).manual_seed(width)
    big, small = _rows(width, dt, limit)
    r = lambda *s: torch.randn(s, generator=g, device=dev()).to(DT[dt])  # noqa: E731
    x, res, dy, bias = r(big, width), r(big, width), r(big, width), r(width)
    keep = torch.from_numpy(oracle.dropout_mask(big * width, 0.3, 1, 2)).to(dev()).reshape(big, width)
    ops = {"bdr_fwd": (lambda x, res, dy, p: L.lsq_bias_dropout_residual_fwd(x, bias, res, p, 1, 2), None),
           "bdr_bwd": (lambda x, res, dy, p: L.lsq_bias_dropout_residual_bwd(dy, p, 1, 2)[0], lambda p: L.lsq_bias_dropout_residual_bwd(dy, p, 1, 2)[1])}
    for act in ("relu", "gelu"):
        ops[act + "_fwd"] = (lambda x, res, dy, p, a=act: L.lsq_bias_act_dropout_fwd(x, bias, a, p, 1, 2), None)
        ops[act + "_bwd"] = (lambda x, res, dy, p, a=act: L.lsq_bias_act_dropout_bwd(dy, x, bias, a, p, 1, 2)[0],
                             lambda p, a=act: L.lsq_bias_act_dropout_bwd(dy, x, bias, a, p, 1, 2)[1])
    for name, (call, sums) in ops.items():
        out = {p: call(x, res, dy, p) for p in (0.0, 0.3)}
        for p in out:
            assert torch.equal(out[p][:small], call(x[:small], res[:small], dy[:small], p)), (name, p)
        assert torch.equal(out[0.0][-small:], call(x[-small:], res[-small:], dy[-small:], 0.0)), name
        # o = r + k z (r the residual, else 0) against r + k (o0 - r): a rounding of o0 that grows by 1 / (1 - p), one of o, and in fp32 those of z and k
        r0, o0, k = (res.double() if name == "bdr_fwd" else 0.0), out[0.0].double(), keep.double() / 0.7
        ref, eps = r0 + k * (o0 - r0), {"f16": 1.01 * 2.0 ** -11, "f32": 2.0 ** -22}[dt]
        err = (out[0.3].double() - ref).abs() - eps * (o0.abs() / 0.7 + ref.abs()) - (2.0 ** -23 if dt == "f16" else 2.0 ** -22)       # (z, and subnormal halves)
        assert err.max() <= 0, (name, float(err.max()))
        if sums is not None:
            for p in out:                      # fp32 sums of what is rounded to `dt` when stored: a rounding per row, of either sign, within half an ulp
                want, rms = out[p].double().sum(0), out[p].double().square().mean().sqrt()
                assert (sums(p).double() - want).norm() <= {"f16": 2.0 ** -11, "f32": 1e-5}[dt] * rms * (big * width) ** 0.5, (name, p)


@pytest.mark.parametrize("limit", LIMITS)
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("heads,head_dim,parts", [(8, 64, 3), (5, 128, 1), (7, 80, 2), (9, 64, 1)])
def test_heads(heads, head_dim, parts, dt, limit):
    say(f"[cached loads] heads {heads} x {head_dim} x {parts} {dt} about {limit}")
    g = torch.Generator(device=dev()).manual_seed(heads)
    ln, hidden = 33, heads * head_dim
    big = limit // (ln * hidden * DT[dt].itemsize) + 2
    small = max(1, big // (2 * parts))
    r = lambda *s: torch.randn(s, generator=g, device=dev()).to(DT[dt])  # noqa: E731
    x, bias = r(big * ln, parts * hidden), r(parts * hidden)
    for b in (None, bias):
        for whole, part in zip(L.lsq_split_heads_fwd(x, b, big, ln, heads, head_dim, parts), L.lsq_split_heads_fwd(x[:small * ln], b, small, ln, heads, head_dim, parts)):
            assert whole is part is None or torch.equal(whole[:small], part)
        for whole, part in zip(L.lsq_split_heads_fwd(x, b, big, ln, heads, head_dim, parts), L.lsq_split_heads_fwd(x[-small * ln:], b, small, ln, heads, head_dim, parts)):
            assert whole is part is None or torch.equal(whole[-small:], part)
    d = [r(big, heads, ln, head_dim) for _ in range(parts)]
    din, dbias = L.lsq_split_heads_bwd(d, big, ln, heads, head_dim)
    assert torch.equal(din[:small * ln], L.lsq_split_heads_bwd([t[:small].contiguous() for t in d], small, ln, heads, head_dim)[0])
    assert torch.equal(din[-small * ln:], L.lsq_split_heads_bwd([t[-small:].contiguous() for t in d], small, ln, heads, head_dim)[0])
    ref = din.double().sum(0)                  # fp32 sums of `rows` normal values: well within 1e-5 of their 2-norm
    assert (dbias.double() - ref).norm() <= 1e-5 * (din.shape[0] ** 0.5) * ref.shape[0] ** 0.5
    assert torch.equal(L.lsq_merge_heads_fwd(d[0])[:small * ln], L.lsq_merge_heads_fwd(d[0][:small].contiguous()))
    assert torch.equal(L.lsq_merge_heads_fwd(d[0])[-small * ln:], L.lsq_merge_heads_fwd(d[0][-small:].contiguous()))


@pytest.mark.parametrize("limit", LIMITS[:1])
@pytest.mark.parametrize("dt", ["f16", "f32"])
def test_padding(dt, limit):
    say(f"[cached loads] padding {dt} about {limit}")
    g = torch.Generator(device=dev()).manual_seed(3)
    ln, hidden = 40, 520
    big = limit // (ln * hidden * DT[dt].itemsize) + 3
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
