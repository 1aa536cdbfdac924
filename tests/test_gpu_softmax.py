"""GPU parity: masked attention softmax forward / backward through the C-ABI against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2110_05722_amd as L
from tests._util import assert_close_store, dev, say, to_np64
from workloads import CONFIGS, attention_tensors, device_normal, encode, from_torch, to_torch

pytestmark = pytest.mark.gpu

# (batch, heads, q_len, k_len, mask, p_attn); mask in {"none", "pad", "causal", "pad+causal"}
CASES = [
    (8, 8, 64, 64, "pad", 0.0), (8, 8, 64, 64, "pad+causal", 0.0),            # config 1
    (128, 8, 32, 32, "pad", 0.0), (128, 8, 32, 32, "pad+causal", 0.0),        # config 2: enc self, dec self
    (64, 16, 128, 128, "pad", 0.1), (64, 16, 128, 128, "pad+causal", 0.1),    # config 3 with attention dropout
    (2, 16, 512, 512, "none", 0.0),                                           # config 4 shape (2 of 16 batches)
    (1, 20, 1024, 1024, "causal", 0.0),                                       # config 5 shape (1 of 8 batches)
    (3, 2, 5, 8, "pad", 0.25), (3, 2, 16, 16, "pad+causal", 0.25),            # 1 and 2 lanes per row
    (2, 3, 50, 50, "pad", 0.1), (2, 3, 33, 33, "pad+causal", 0.2),            # odd lengths
    (2, 2, 7, 24, "causal", 0.0), (2, 2, 24, 40, "pad+causal", 0.1),          # q_len != k_len, end-aligned
    (2, 2, 9, 256, "pad", 0.0), (2, 2, 9, 768, "pad", 0.1), (1, 2, 5, 1536, "causal", 0.0),
    (1, 2, 3, 2048, "pad", 0.1), (1, 1, 3, 4096, "pad", 0.1), (1, 1, 2, 1, "none", 0.0),
    # long rows: one workgroup per row (2048 < k_len <= 16384), and the fallback beyond
    (2, 1, 4, 2056, "pad", 0.1), (1, 2, 3, 8192, "pad+causal", 0.1), (1, 1, 2, 16384, "pad", 0.0),
    (1, 1, 2, 16392, "pad", 0.1), (2, 1, 5, 4099, "pad+causal", 0.1),
    # lengths that are not a multiple of 8, over both forms of such rows (registers and LDS)
    (3, 2, 5, 7, "pad", 0.25), (3, 2, 9, 9, "pad+causal", 0.1), (4, 2, 17, 17, "pad", 0.1), (2, 2, 31, 33, "pad+causal", 0.0),
    (2, 2, 63, 63, "pad", 0.1), (2, 2, 65, 65, "causal", 0.1), (64, 4, 100, 100, "pad", 0.1), (2, 3, 127, 127, "pad+causal", 0.1),
    (2, 2, 20, 129, "pad", 0.0), (2, 2, 12, 255, "pad", 0.1), (2, 1, 9, 500, "pad", 0.1), (2, 1, 6, 513, "causal", 0.1),
    (1, 2, 5, 1001, "pad", 0.1), (1, 2, 4, 1025, "pad", 0.0), (1, 1, 3, 2047, "pad", 0.1), (1, 1, 3, 2049, "pad", 0.1),
    (1, 3, 1, 3, "none", 0.5),
]


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("B,N,Lq,Lk,mask,p", CASES)
def test_softmax_fwd_bwd(B, N, Lq, Lk, mask, p, dt):
    if dt == "f32" and B * N * Lq * Lk > 1 << 21:
        pytest.skip("fp32 storage is exercised on the small shapes only")
    say(f"[softmax] B={B} N={N} Lq={Lq} Lk={Lk} mask={mask} p={p} dt={dt}")
    cfg = next((c for c in CONFIGS if c.batch == B and c.max_len == Lk), CONFIGS[0])
    t = attention_tensors(cfg, dt, batch=B, heads=N, q_len=Lq, k_len=Lk, stream=300 + Lk)
    key_len = t["key_len"] if "pad" in mask else None
    causal = "causal" in mask
    scale = 1.0 / np.sqrt(64.0)
    seed, offset = 4321, Lk
    d = dev()
    x, dy = to_torch(t["x"], dt, d), to_torch(t["dy"], dt, d)
    kl = None if key_len is None else torch.from_numpy(key_len).to(d)
    y, yd = L.lsq_softmax_fwd(x, kl, causal, scale, p, seed, offset)
    ry, ryd = oracle.softmax_fwd(t["x"], key_len, causal, scale, dt, p, seed, offset)
    assert_close_store(y, ry, dt, "y", f32_floor=1e-7)
    # positions outside the allowed set are exactly +0 (bit pattern), not merely small
    masked = ry == 0.0
    ybits = from_torch(y, dt)
    assert not ybits.reshape(ry.shape)[masked].view(np.uint16 if dt != "f32" else np.uint32).any()
    if p > 0:
        assert_close_store(yd, ryd, dt, "y_drop", f32_floor=1e-7)
        # the dropped set is bit-exact
        assert np.array_equal(to_np64(yd, dt) == 0, ryd == 0)
    # backward takes the y the GPU stored, on both sides
    ystored = from_torch(y, dt)
    dx = L.lsq_softmax_bwd(dy, y, kl, causal, scale, p, seed, offset)
    rdx = oracle.softmax_bwd(t["dy"], ystored, key_len, causal, scale, dt, p, seed, offset)
    assert_close_store(dx, rdx, dt, "dx", f32_floor=1e-7)
    assert not from_torch(dx, dt).reshape(ry.shape)[masked].view(np.uint16 if dt != "f32" else np.uint32).any()
    # in place: dx over dy
    dyc = dy.clone()
    dx2 = L.lsq_softmax_bwd(dyc, y, kl, causal, scale, p, seed, offset, dx=dyc)
    assert torch.equal(dx, dx2)


@pytest.mark.parametrize("scale", [-0.125, 0.0, 3.0])
@pytest.mark.parametrize("B,N,Lq,Lk,mask,p", [(2, 2, 9, 128, "pad", 0.1), (1, 2, 5, 1024, "causal", 0.0), (2, 1, 3, 2048, "pad+causal", 0.1),
                                              (1, 1, 3, 4096, "pad", 0.1)])
def test_softmax_other_scales(B, N, Lq, Lk, mask, p, scale):
    """The scale is any float by contract: negative and zero scales (rows of whole packs up to 2048 keys take
    another kernel for them), and a large one that spreads the exponents."""
    say(f"[softmax] scale={scale} B={B} N={N} Lq={Lq} Lk={Lk} mask={mask} p={p}")
    dt = "f16"
    t = attention_tensors(CONFIGS[0], dt, batch=B, heads=N, q_len=Lq, k_len=Lk, stream=900 + Lk)
    key_len = t["key_len"] if "pad" in mask else None
    causal = "causal" in mask
    d = dev()
    x, dy = to_torch(t["x"], dt, d), to_torch(t["dy"], dt, d)
    kl = None if key_len is None else torch.from_numpy(key_len).to(d)
    y, yd = L.lsq_softmax_fwd(x, kl, causal, scale, p, 77, 5)
    ry, ryd = oracle.softmax_fwd(t["x"], key_len, causal, scale, dt, p, 77, 5)
    assert_close_store(y, ry, dt, "y", f32_floor=1e-7)
    if p > 0:
        assert_close_store(yd, ryd, dt, "y_drop", f32_floor=1e-7)
    dx = L.lsq_softmax_bwd(dy, y, kl, causal, scale, p, 77, 5)
    rdx = oracle.softmax_bwd(t["dy"], from_torch(y, dt), key_len, causal, scale, dt, p, 77, 5)
    assert_close_store(dx, rdx, dt, "dx", f32_floor=1e-7)


def test_softmax_key_len_edge_values():
    say("[softmax] key_len 0, 1, beyond k_len, negative")
    d, dt = dev(), "f16"
    t = attention_tensors(CONFIGS[0], dt, batch=4, heads=2, q_len=16, k_len=64, stream=399)
    key_len = np.array([0, 1, 100, -3], np.int32)
    x = to_torch(t["x"], dt, d)
    y, _ = L.lsq_softmax_fwd(x, torch.from_numpy(key_len).to(d), False, 1.0)
    ry, _ = oracle.softmax_fwd(t["x"], key_len, False, 1.0, dt)
    assert_close_store(y, ry, dt, "y")
    yy = y.float().cpu().numpy()
    assert (yy[0] == 0).all() and (yy[3] == 0).all() and (yy[1, :, :, 0] == 1).all() and np.isfinite(yy).all()
    assert np.allclose(yy[2].sum(-1), 1, atol=2e-3)


@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_softmax_full_size_gpt2_large(dt):
    """Config 5 at full size, the launch the benchmark times; the oracle checks two whole batches."""
    say(f"[softmax] full size [8,20,1024,1024] causal dt={dt}")
    d = dev()
    B, N, Lq = 8, 20, 1024
    x = device_normal((B, N, Lq, Lq), 1.0, dt, seed=4, device=d)
    dy = device_normal((B, N, Lq, Lq), 1.0, dt, seed=5, device=d)
    scale = 0.125
    y, _ = L.lsq_softmax_fwd(x, None, True, scale)
    dx = L.lsq_softmax_bwd(dy, y, None, True, scale)
    for b in (0, 7):
        ry, _ = oracle.softmax_fwd(from_torch(x[b:b + 1], dt), None, True, scale, dt)
        assert_close_store(y[b:b + 1], ry, dt, f"y[{b}]")
        rdx = oracle.softmax_bwd(from_torch(dy[b:b + 1], dt), from_torch(y[b:b + 1], dt), None, True, scale, dt)
        assert_close_store(dx[b:b + 1], rdx, dt, f"dx[{b}]")
    # properties over the whole tensor: rows sum to 1, the strict upper triangle is exactly zero
    s = y.float().sum(-1)
    assert torch.all((s - 1).abs() < (2e-2 if dt == "bf16" else 4e-3))
    upper = torch.triu(torch.ones(Lq, Lq, dtype=torch.bool, device=d), diagonal=1)
    assert not y[:, :, upper].any() and not dx[:, :, upper].any()


def test_softmax_full_size_transformer_big_with_dropout():
    """Config 3 at full size with attention dropout and both masks."""
    say("[softmax] full size [64,16,128,128] pad+causal p=0.1")
    d, dt = dev(), "f16"
    cfg = CONFIGS[2]
    t = attention_tensors(cfg, dt)
    x, dy = to_torch(t["x"], dt, d), to_torch(t["dy"], dt, d)
    kl = torch.from_numpy(t["key_len"]).to(d)
    y, yd = L.lsq_softmax_fwd(x, kl, True, 0.125, cfg.p_attn, cfg.philox_seed, 9)
    ry, ryd = oracle.softmax_fwd(t["x"], t["key_len"], True, 0.125, dt, cfg.p_attn, cfg.philox_seed, 9)
    assert_close_store(y, ry, dt, "y")
    assert_close_store(yd, ryd, dt, "y_drop")
    assert np.array_equal(to_np64(yd, dt) == 0, ryd == 0)
    dx = L.lsq_softmax_bwd(dy, y, kl, True, 0.125, cfg.p_attn, cfg.philox_seed, 9)
    rdx = oracle.softmax_bwd(t["dy"], from_torch(y, dt), t["key_len"], True, 0.125, dt, cfg.p_attn, cfg.philox_seed, 9)
    assert_close_store(dx, rdx, dt, "dx")


# rows that are not whole packs: both sides of every bucket edge (a row of k keys touches up to (k + 14) / 8 packs for odd
# k, fewer for k = 2 or 4 mod 8), one row, and a tensor whose last pack is cut short
RAGGED = [2, 9, 10, 12, 15, 25, 26, 28, 57, 58, 63, 66, 100, 121, 122, 124, 185, 187, 249, 251, 377, 379, 505, 507, 761, 763, 1017, 1019, 1529, 1531, 2041, 2043,
          4089, 4091, 8185, 8187, 16377, 16379]


@pytest.mark.parametrize("scale,p", [(0.125, 0.1), (-0.5, 0.0)])
@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("Lk", RAGGED)
def test_softmax_ragged_rows(Lk, dt, scale, p):
    say(f"[softmax] ragged rows Lk={Lk} dt={dt} scale={scale} p={p}")
    d = dev()
    B, N, Lq = 3, 1, 3 if Lk > 1000 else 11
    t = attention_tensors(CONFIGS[0], dt, batch=B, heads=N, q_len=Lq, k_len=Lk, stream=1200 + Lk)
    key_len, query_len = np.array([Lk, max(1, Lk // 3), max(1, Lk - 1)], np.int32), np.array([Lq, 1, Lq - 1], np.int32)
    x, dy = to_torch(t["x"], dt, d), to_torch(t["dy"], dt, d)
    kl, ql = torch.from_numpy(key_len).to(d), torch.from_numpy(query_len).to(d)
    ry, ryd = oracle.softmax_fwd(t["x"], key_len, False, scale, dt, p, 11, 3, query_len=query_len)
    # what lies outside the mask never counts, whatever it holds
    off = torch.arange(Lk, device=d)[None, None, None, :] >= kl[:, None, None, None]
    off = off | (torch.arange(Lq, device=d)[None, None, :, None] >= ql[:, None, None, None])
    x, dy = x.masked_fill(off, float("nan")), dy.masked_fill(off, float("nan"))
    y, yd = L.lsq_softmax_varlen_fwd(x, kl, ql, False, scale, p, 11, 3)
    assert_close_store(y, ry, dt, "y", f32_floor=1e-7)
    assert not y[off].any()
    if p > 0:
        assert_close_store(yd, ryd, dt, "y_drop", f32_floor=1e-7)
        assert np.array_equal(to_np64(yd, dt) == 0, ryd == 0)
    dx = L.lsq_softmax_varlen_bwd(dy, y, kl, ql, False, scale, p, 11, 3)
    rdx = oracle.softmax_bwd(t["dy"], from_torch(y, dt), key_len, False, scale, dt, p, 11, 3, query_len=query_len)
    assert_close_store(dx, rdx, dt, "dx", f32_floor=1e-7)
    # in place, forward and backward
    assert torch.equal(L.lsq_softmax_varlen_fwd(x, kl, ql, False, scale, p, 11, 3, y=x)[0], y)
    assert torch.equal(L.lsq_softmax_varlen_bwd(dy, y, kl, ql, False, scale, p, 11, 3, dx=dy), dx)


# every path of the dispatch: a lane's own pack, several lanes, a whole wave, a workgroup per row, the element-strided kernel beyond;
# rows of whole packs and others
@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("Lk", [8, 64, 1024, 2056, 16392, 5, 14, 26, 45, 63, 113, 180, 201, 1001, 2039, 2047, 4099, 16379])
def test_softmax_nonfinite_values_stay_inside_the_mask(Lk, dt):
    """Infinities and NaN inside the allowed set (a mixed-precision overflow step) spoil their row's allowed positions only:
    positions outside the mask are +0, dropped ones of y_drop are 0, and other rows do not change by a bit."""
    say(f"[softmax] non-finite values inside the mask Lk={Lk} dt={dt}")
    d, p, seed, offset = dev(), 0.25, 21, 8
    B, N, Lq = 2, 1, 5
    t = attention_tensors(CONFIGS[0], dt, batch=B, heads=N, q_len=Lq, k_len=Lk, stream=1300 + Lk)
    kl = torch.tensor([max(2, Lk // 2), max(3, Lk - 3)], dtype=torch.int32, device=d)
    x, dy = to_torch(t["x"], dt, d), to_torch(t["dy"], dt, d)
    a = (kl, None, False, 0.125, p, seed, offset)
    y, yd = L.lsq_softmax_varlen_fwd(x, *a)
    dx = L.lsq_softmax_varlen_bwd(dy, y, *a)
    beyond = (torch.arange(Lk, device=d)[None, None, None, :] >= kl[:, None, None, None]).expand(B, N, Lq, Lk)
    keep = torch.from_numpy(oracle.dropout_mask(B * N * Lq * Lk, p, seed, offset).reshape(B, N, Lq, Lk) != 0).to(d)
    inside = ~beyond

    def zero_bits(v, where):
        return not v[where].view(torch.int16 if dt != "f32" else torch.int32).any()

    xb = x.clone()
    xb[0, 0, 0, 0], xb[0, 0, 2, 1], xb[1, 0, 3, 1] = float("nan"), float("inf"), float("-inf")   # the last is an ordinary score
    xb[1, 0, 1] = float("-inf")
    yb, ydb = L.lsq_softmax_varlen_fwd(xb, *a)
    for v, w in ((yb, y), (ydb, yd)):
        assert zero_bits(v, beyond)
        for b, i in ((0, 1), (0, 3), (0, 4), (1, 0), (1, 2), (1, 4)):
            assert torch.equal(v[b, 0, i], w[b, 0, i])
    assert zero_bits(ydb, ~keep)
    for b, i in ((0, 0), (0, 2), (1, 1)):
        assert yb[b, 0, i, 0].isnan()
    assert yb[1, 0, 3].isfinite().all() and yb[1, 0, 3, 1] == 0

    g = dy.clone()
    hit = []                                             # (batch, row) with an infinity or a NaN at a kept allowed position
    for b, i, v in ((0, 0, "inf"), (0, 2, "nan"), (1, 1, "-inf"), (1, 4, "nan")):
        at = (keep & inside)[b, 0, i].nonzero().flatten()
        at = at[y[b, 0, i][at] > 0]
        if len(at):
            g[b, 0, i, at[0]] = float(v)
            hit.append((b, i))
    if Lk % 8 and Lk < 2041:
        g = g.masked_fill(~keep, float("inf"))           # dy where the forward dropped (the other paths multiply it by a factor of 0)
    dxb = L.lsq_softmax_varlen_bwd(g, y, *a)
    assert zero_bits(dxb, beyond)
    for b in range(B):
        for i in range(Lq):
            if (b, i) in hit:
                assert not dxb[b, 0, i].isfinite().all()
            else:
                assert torch.equal(dxb[b, 0, i], dx[b, 0, i])


# the lines between the register and the LDS form of rows that are not whole packs: each LDS shape and direction, at the sizes and masks
# that send a call there (whole rows of the workgroup's range, a cut last workgroup, tensors beyond 256 MB)
LDS_ROWS = [("f32", 3, 2, 7, 7, "none", 0.1), ("f32", 5, 2, 13, 12, "none", 0.0), ("f32", 3, 2, 17, 17, "none", 0.0), ("f32", 2, 3, 33, 28, "pad", 0.1),
            ("f16", 4, 3, 15, 15, "none", 0.1), ("f16", 4, 3, 29, 29, "causal", 0.0), ("f16", 3, 2, 45, 45, "pad", 0.1), ("f16", 140, 8, 63, 63, "causal", 0.0),
            ("f32", 500, 8, 33, 34, "none", 0.0), ("f32", 2, 3, 20, 70, "none", 0.0), ("f16", 2, 3, 20, 127, "none", 0.1), ("f16", 2, 3, 20, 255, "causal", 0.1),
            ("f16", 9, 8, 255, 255, "none", 0.0), ("f16", 2, 2, 9, 511, "none", 0.1), ("f16", 2, 2, 9, 150, "pad", 0.1), ("f32", 2, 2, 9, 150, "none", 0.1),
            ("f32", 4, 6, 7000, 134, "none", 0.0), ("f16", 2, 4, 56000, 100, "none", 0.0), ("f16", 2, 4, 56000, 101, "none", 0.1)]


@pytest.mark.parametrize("dt,B,N,Lq,Lk,mask,p", LDS_ROWS)
def test_softmax_rows_through_lds(dt, B, N, Lq, Lk, mask, p):
    say(f"[softmax] rows through LDS {dt} {B}x{N}x{Lq}x{Lk} mask={mask} p={p}")
    d, scale, causal = dev(), 0.125, mask == "causal"
    x, dy = (device_normal((B, N, Lq, Lk), 1.0, dt, seed=s, device=d) for s in (1, 2))
    key_len = np.array([max(1, Lk * (b + 1) // B) for b in range(B)], np.int32) if mask == "pad" else None
    kl = None if key_len is None else torch.from_numpy(key_len).to(d)
    y, yd = L.lsq_softmax_fwd(x, kl, causal, scale, p, 5, 6)
    dx = L.lsq_softmax_bwd(dy, y, kl, causal, scale, p, 5, 6)
    n = x.numel()
    few = n > 1 << 20                                                # the first and the last sentences' first head only
    for b in (range(0, B, max(1, B - 1)) if few else [slice(None)]):
        at = np.s_[b:b + 1, :1] if few else np.s_[:, :]
        lens = None if key_len is None else key_len[at[0]]
        e0 = b * N * Lq * Lk if few else 0
        ry, ryd = oracle.softmax_fwd(from_torch(x[at].contiguous(), dt), lens, causal, scale, dt, p, 5, 6, e0=e0)
        assert_close_store(y[at], ry, dt, "y", f32_floor=1e-7)
        if p > 0:
            assert_close_store(yd[at], ryd, dt, "y_drop", f32_floor=1e-7)
        rdx = oracle.softmax_bwd(from_torch(dy[at].contiguous(), dt), from_torch(y[at].contiguous(), dt), lens, causal, scale, dt, p, 5, 6, e0=e0)
        assert_close_store(dx[at], rdx, dt, "dx", f32_floor=1e-7)


# waves whose rows are all empty leave early and write their rows as one range of zeros: rows of every lane count, whole packs and not,
# ranges that begin and end anywhere in a pack, an empty sentence beside a full one, rows above a causal mask's first key
@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Lq,Lk", [(70, 3), (70, 8), (66, 13), (70, 24), (131, 31), (70, 64), (67, 113), (70, 128), (41, 130), (37, 256), (33, 301), (19, 512), (19, 701),
                                   (17, 1000), (70, 9)])
def test_softmax_rows_of_padded_queries(Lq, Lk, causal, dt):
    say(f"[softmax] padded queries {Lq} x {Lk} causal={causal} {dt}")
    B, N, p, d = 5, 3, 0.2, dev()
    r = np.random.default_rng(Lq * 1000 + Lk)
    xs, dys = (encode(r.standard_normal((B, N, Lq, Lk), dtype=np.float32), dt) for _ in range(2))
    klen, qlen = np.array([Lk, 1, Lk // 2, Lk, 0], np.int32), np.array([1, Lq, 0, Lq // 2, Lq], np.int32)
    kl, ql = torch.from_numpy(klen).to(d), torch.from_numpy(qlen).to(d)
    y, yd = L.lsq_softmax_varlen_fwd(to_torch(xs, dt, d), kl, ql, causal, 0.4, p, 3, 5)
    ry, ryd = oracle.softmax_fwd(xs, klen, causal, 0.4, dt, p, 3, 5, query_len=qlen)
    assert_close_store(y, ry, dt, "y")
    assert_close_store(yd, ryd, dt, "y_drop")
    dx = L.lsq_softmax_varlen_bwd(to_torch(dys, dt, d), y, kl, ql, causal, 0.4, p, 3, 5)
    assert_close_store(dx, oracle.softmax_bwd(dys, from_torch(y, dt).reshape(ry.shape), klen, causal, 0.4, dt, p, 3, 5, query_len=qlen), dt, "dx")
    for t in (y, yd, dx):                                   # +0 to the bit where nothing is allowed, and nothing is read there
        t = t.view(B, N, Lq, Lk)
        for b in range(B):
            assert not t[b, :, qlen[b]:].view(torch.int32 if dt == "f32" else torch.int16).any()
    spoilt = to_torch(xs, dt, d).view(B, N, Lq, Lk).clone()
    for b in range(B):
        spoilt[b, :, qlen[b]:] = float("nan")
    assert torch.equal(L.lsq_softmax_varlen_fwd(spoilt, kl, ql, causal, 0.4, 0.0)[0], L.lsq_softmax_varlen_fwd(to_torch(xs, dt, d).view(B, N, Lq, Lk), kl, ql, causal, 0.4, 0.0)[0])


# the lines of the loads behind the limit and of the waves that leave (128 and 1024 bytes, 640, 1024 and 1536 keys, more queries than keys), both sides
@pytest.mark.parametrize("dt", ["f16", "f32"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Lq,Lk", [(66, 16), (66, 32), (32, 32), (40, 40), (66, 40), (30, 40), (66, 65), (35, 248), (35, 255), (35, 257), (21, 504), (21, 520), (21, 639),
                                   (21, 641), (19, 1023), (19, 1024), (19, 1032), (19, 1536), (19, 1537)])
def test_softmax_padded_queries_at_the_lines(Lq, Lk, causal, dt):
    test_softmax_rows_of_padded_queries(Lq, Lk, causal, dt)
