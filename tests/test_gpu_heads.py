"""GPU parity: head split / merge through the C-ABI against the CPU oracle.  Pure moves are bit-exact."""
import numpy as np
import pytest
import torch

import oracle
import paper_2110_05722_amd as L
from tests._util import assert_close_f32, assert_close_store, dev, say
from workloads import decode, encode, from_torch, to_torch

pytestmark = pytest.mark.gpu

# (batch, len, heads, head_dim, parts)
CASES = [(8, 64, 8, 64, 3), (128, 32, 8, 64, 3), (16, 128, 16, 64, 3), (2, 512, 16, 64, 3), (1, 1024, 20, 64, 3),
         (3, 50, 12, 64, 1), (2, 33, 5, 8, 2), (2, 7, 3, 24, 3), (3, 5, 2, 5, 3), (1, 1, 1, 1, 1), (2, 9, 4, 128, 2)]


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("B,Ln,N,D,parts", CASES)
def test_split_heads_fwd_bwd(B, Ln, N, D, parts, dt):
    if dt == "f32" and B * Ln * N * D * parts > 1 << 21:
        pytest.skip("fp32 storage is exercised on the small shapes only")
    split_heads_against_the_oracle(B, Ln, N, D, parts, dt)


def split_heads_against_the_oracle(B, Ln, N, D, parts, dt):
    say(f"[heads] B={B} L={Ln} N={N} D={D} parts={parts} dt={dt}")
    d = dev()
    r = np.random.default_rng(B * 1000 + Ln + D)
    H = N * D
    xs = encode(r.standard_normal((B * Ln, parts * H), dtype=np.float32), dt)
    bs = encode(r.standard_normal(parts * H, dtype=np.float32) * 0.1, dt)
    x, bias = to_torch(xs, dt, d), to_torch(bs, dt, d)
    outs = L.lsq_split_heads_fwd(x, bias, B, Ln, N, D, parts)
    refs = oracle.split_heads_fwd(xs, bs, B, Ln, N, D, parts, dt)
    for k in range(parts):
        assert_close_store(outs[k], refs[k], dt, f"out{k}")
    # without bias: bit-exact against the oracle's (exact) permutation of the stored values
    outs_nb = L.lsq_split_heads_fwd(x, None, B, Ln, N, D, parts)
    refs_nb = oracle.split_heads_fwd(xs, None, B, Ln, N, D, parts, dt)
    for k in range(parts):
        assert np.array_equal(decode(from_torch(outs_nb[k], dt), dt).reshape(refs_nb[k].shape), refs_nb[k])
    # backward: gather + column sums
    gs = [encode(r.standard_normal((B, N, Ln, D), dtype=np.float32), dt) for _ in range(parts)]
    grads = [to_torch(g, dt, d) for g in gs]
    din, dbias = L.lsq_split_heads_bwd(grads, B, Ln, N, D)
    rdin, rdb = oracle.split_heads_bwd(gs, B, Ln, N, D, dt)
    assert np.array_equal(decode(from_torch(din, dt), dt).reshape(rdin.shape), rdin)
    assert_close_f32(dbias, rdb, "dbias", floor=1e-6 * np.sqrt(B * Ln) * 4)
    din2, none = L.lsq_split_heads_bwd(grads, B, Ln, N, D, want_dbias=False)
    assert none is None and torch.equal(din, din2)


@pytest.mark.parametrize("B,Ln,N,D", [(8, 1024, 20, 64), (64, 128, 16, 64), (2, 9, 3, 5)])
def test_merge_heads_round_trip(B, Ln, N, D):
    say(f"[heads] merge B={B} L={Ln} N={N} D={D}")
    d = dev()
    x = torch.randn((B, N, Ln, D), device=d).to(torch.float16)
    out = L.lsq_merge_heads_fwd(x)
    assert torch.equal(out, x.permute(0, 2, 1, 3).reshape(B * Ln, N * D))      # index work: bit-exact
    back = L.lsq_merge_heads_bwd(out, B, Ln, N, D)
    assert torch.equal(back, x)
    ref, _ = oracle.split_heads_bwd([from_torch(x, "f16")], B, Ln, N, D, "f16", want_dbias=False)
    assert np.array_equal(out.float().cpu().numpy().astype(np.float64), ref)


def test_heads_empty():
    d = dev()
    x = torch.empty((0, 3 * 64), dtype=torch.float16, device=d)
    outs = L.lsq_split_heads_fwd(x, None, 0, 5, 1, 64, 3)
    din, dbias = L.lsq_split_heads_bwd(outs, 0, 5, 1, 64)
    torch.cuda.synchronize()
    assert din.numel() == 0 and dbias.abs().sum().item() == 0


# the column sums' rows per partial row in fp32 on both sides of 3.2 M elements
@pytest.mark.parametrize("rows", [1666, 1667, 2048])
def test_split_heads_bwd_rows_per_partial_row(rows):
    split_heads_against_the_oracle(1, rows, 8, 80, 3, "f32")
