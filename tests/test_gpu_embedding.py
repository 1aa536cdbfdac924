"""GPU parity: embedding forward / backward through the C-ABI against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2110_05722_amd as L
from tests._util import LP_TOL, assert_close_store, dev, say
from workloads import decode, encode, from_torch, to_torch

pytestmark = pytest.mark.gpu
PAD = 1

# (batch, len, vocab, hidden, p)
CASES = [(8, 64, 8000, 512, 0.1), (128, 32, 32768, 512, 0.1), (16, 128, 4096, 1024, 0.3), (4, 512, 30522, 1024, 0.1),
         (2, 1024, 50257, 1280, 0.1), (3, 50, 97, 768, 0.0), (5, 7, 11, 8, 0.25), (2, 9, 13, 257, 0.2), (1, 1, 3, 64, 0.1),
         (4, 300, 5, 64, 0.1),
         (40, 520, 1000, 64, 0.1),      # beyond 16384 tokens: the radix-sorted order, two passes
         (36, 512, 100, 16, 0.1), (9, 2048, 70001, 16, 0.1),      # one pass (ids below 256) and three (above 65535)
         (550, 2000, 3000, 8, 0.1),     # 1.1 M tokens: the radix passes with the stand-alone offset scan
         (1, 70000, 500, 8, 0.1),       # one sentence longer than 65535 positions
         (4, 4096, 50257, 8, 0.0)]      # exactly 16384 tokens: the most that the in-LDS sort takes


def _tokens(B, Ln, V, rng):
    # Zipf-like ids so that some tokens repeat hundreds of times, the tail of each sentence padded
    tok = np.minimum((rng.pareto(1.1, size=(B, Ln)) * 3).astype(np.int64) + 2, V - 1).astype(np.int32)
    lens = rng.integers(max(1, Ln // 2), Ln + 1, size=B)
    tok[np.arange(Ln)[None, :] >= lens[:, None]] = PAD
    if B * Ln > 4:
        tok.reshape(-1)[3] = V            # out of range -> padding
        tok.reshape(-1)[2] = V - 1
    return tok


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("B,Ln,V,H,p", CASES)
def test_embedding_fwd_bwd(B, Ln, V, H, p, dt):
    if dt == "f32" and (B * Ln * H > 1 << 21 or V * H > 1 << 23):
        pytest.skip("fp32 storage is exercised on the small shapes only")
    say(f"[embedding] B={B} L={Ln} V={V} H={H} p={p} dt={dt}")
    d = dev()
    rng = np.random.default_rng(B * 7 + Ln + V)
    tok = _tokens(B, Ln, V, rng)
    embs = encode(rng.standard_normal((V, H), dtype=np.float32), dt)
    poss = encode(rng.standard_normal((Ln, H), dtype=np.float32) * 0.5, dt)
    dys = encode(rng.standard_normal((B * Ln, H), dtype=np.float32), dt)
    scale, seed, offset = float(np.sqrt(H)), 31, Ln
    tokens = torch.from_numpy(tok).to(d)
    emb, pos, dy = to_torch(embs, dt, d), to_torch(poss, dt, d), to_torch(dys, dt, d)
    out = L.lsq_embedding_fwd(tokens, emb, pos, PAD, scale, p, seed, offset)
    ref = oracle.embedding_fwd(tok, embs, poss, PAD, scale, p, seed, offset, dt)
    # values reach |scale * 4|: the relative (one ulp) branch of the tolerance is the one that binds
    assert_close_store(out, ref, dt, "out", f32_floor=1e-5)
    assert np.array_equal(decode(from_torch(out, dt), dt).reshape(ref.shape) == 0, ref == 0)

    # backward accumulates into existing gradients
    d0 = encode(rng.standard_normal((V, H), dtype=np.float32) * 0.1, dt)
    p0 = encode(rng.standard_normal((Ln, H), dtype=np.float32) * 0.1, dt)
    demb, dpos = to_torch(d0, dt, d), to_torch(p0, dt, d)
    L.lsq_embedding_bwd(demb, dpos, dy, tokens, PAD, scale, p, seed, offset)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, scale, p, seed, offset, dt)
    # a frequent token sums hundreds of rows of size scale*|dy|: widen the absolute term by the row's own magnitude
    assert_close_store(demb, decode(d0, dt) + inc_e, dt, "demb", f32_floor=1e-4 * scale)
    assert_close_store(dpos, decode(p0, dt) + inc_p, dt, "dpos", f32_floor=1e-4)
    # untouched rows keep their bits (padding row, ids that do not occur)
    flat = tok.reshape(-1)
    used = np.unique(flat[(flat != PAD) & (flat >= 0) & (flat < V)])
    unused = np.setdiff1d(np.arange(V), used)
    assert np.array_equal(from_torch(demb, dt)[unused], d0[unused])
    # run-to-run bit reproducibility (no atomics), and dpos is optional
    demb2 = to_torch(d0, dt, d)
    L.lsq_embedding_bwd(demb2, None, dy, tokens, PAD, scale, p, seed, offset)
    assert torch.equal(demb, demb2)


@pytest.mark.parametrize("kind", ["all padding", "one id everywhere", "all distinct"])
def test_embedding_bwd_degenerate_batches(kind):
    """Batches at the ends of the id distribution: nothing to accumulate, one segment that spans every window of the
    sorted order, and no repeated id at all."""
    say(f"[embedding] degenerate batch: {kind}")
    d, dt = dev(), "f16"
    B, Ln, V, H = 7, 41, 400, 64                   # 287 tokens: a ragged last rank tile and a ragged last window
    rng = np.random.default_rng(17)
    if kind == "all padding":
        tok = np.full((B, Ln), PAD, np.int32)
    elif kind == "one id everywhere":
        tok = np.full((B, Ln), 9, np.int32)
    else:
        tok = (rng.permutation(V - 2)[:B * Ln] + 2).astype(np.int32).reshape(B, Ln)
    dys = encode(rng.standard_normal((B * Ln, H), dtype=np.float32), dt)
    d0 = encode(rng.standard_normal((V, H), dtype=np.float32) * 0.1, dt)
    p0 = encode(rng.standard_normal((Ln, H), dtype=np.float32) * 0.1, dt)
    demb, dpos = to_torch(d0, dt, d), to_torch(p0, dt, d)
    L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), torch.from_numpy(tok).to(d), PAD, 8.0, 0.1, 5, 2)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 8.0, 0.1, 5, 2, dt)
    assert_close_store(demb, decode(d0, dt) + inc_e, dt, "demb", f32_floor=1e-3)
    assert_close_store(dpos, decode(p0, dt) + inc_p, dt, "dpos", f32_floor=1e-4)
    if kind == "all padding":
        assert np.array_equal(from_torch(demb, dt), d0) and np.array_equal(from_torch(dpos, dt), p0)


# the in-LDS sort (64 workgroups, rounds of 256 tokens): one token less than a round and so on up to its largest, on both sides of the
# 8192 tokens that a workgroup holds at once, ids of one, two and three digits, the hand-over to the sort over many workgroups; and
# the position gradient on both sides of 16 sentences
@pytest.mark.parametrize("B,Ln,V", [(1, 63, 255), (1, 64, 256), (1, 255, 300), (1, 257, 300), (3, 341, 65535), (1, 8191, 50257), (1, 8193, 50257), (1, 1024, 65536), (25, 41, 300), (16, 512, 50257),
                                    (17, 482, 70000), (17, 71, 9), (64, 255, 40), (4, 1500, 3), (1, 16384, 50257), (5, 3277, 50257)])
def test_embedding_bwd_token_order(B, Ln, V):
    say(f"[embedding] token order B={B} L={Ln} V={V}")
    d, dt, H = dev(), "f16", 24
    rng = np.random.default_rng(B + Ln + V)
    tok = _tokens(B, Ln, V, rng)
    dys = encode(rng.standard_normal((B * Ln, H), dtype=np.float32) * 0.05, dt)
    d0, p0 = encode(np.zeros((V, H), np.float32), dt), encode(np.zeros((Ln, H), np.float32), dt)
    demb, dpos = to_torch(d0, dt, d), to_torch(p0, dt, d)
    L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), torch.from_numpy(tok).to(d), PAD, 2.0, 0.1, 3, 7)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 2.0, 0.1, 3, 7, dt)
    assert_close_store(demb, inc_e, dt, "demb")
    assert_close_store(dpos, inc_p, dt, "dpos")


# rows that are not whole packs: one column, less than a pack, a pack and a bit, both sides of a 64-pack column block; every
# alignment of a row start (odd, 2 and 4 mod 8), segments that cross windows, and the last rows of each tensor
@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("H", [1, 7, 9, 100, 511, 514, 1001, 1441])
def test_embedding_rows_of_any_length(H, dt):
    say(f"[embedding] rows of any length H={H} dt={dt}")
    d, B, Ln, V = dev(), 19, 23, 40                     # the forward of 437 tokens takes one element per thread up to 915 columns
    rng = np.random.default_rng(H)
    tok = _tokens(B, Ln, V, rng)
    tok[-1, -1], tok[0, 0] = V - 1, 2
    mk = lambda shape, std: encode(rng.standard_normal(shape, dtype=np.float32) * np.float32(std), dt)  # noqa: E731
    embs, poss, dys, d0, p0 = mk((V, H), 1), mk((Ln, H), 0.5), mk((B * Ln, H), 0.05), mk((V, H), 0.1), mk((Ln, H), 0.1)
    t = torch.from_numpy(tok).to(d)
    # every tensor ends where its allocation's neighbour begins: guard words behind it must keep their value
    def guarded(a):
        flat = to_torch(a, dt, d).reshape(-1)
        buf = torch.full((flat.numel() + 64,), 7.0, dtype=flat.dtype, device=d)
        buf[:flat.numel()] = flat
        return buf, buf[:flat.numel()].view(a.shape)
    bout, out = guarded(np.zeros_like(dys))
    L.lsq_embedding_fwd(t, to_torch(embs, dt, d), to_torch(poss, dt, d), PAD, 2.0, 0.2, 9, 4, out=out)
    ref = oracle.embedding_fwd(tok, embs, poss, PAD, 2.0, 0.2, 9, 4, dt)
    assert_close_store(out, ref, dt, "out", f32_floor=1e-5)
    assert np.array_equal(decode(from_torch(out, dt), dt).reshape(ref.shape) == 0, ref == 0)
    (be, demb), (bp, dpos) = guarded(d0), guarded(p0)
    L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), t, PAD, 2.0, 0.2, 9, 4)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 2.0, 0.2, 9, 4, dt)
    assert_close_store(demb, decode(d0, dt).reshape(V, H) + inc_e, dt, "demb", f32_floor=1e-5)
    assert_close_store(dpos, decode(p0, dt).reshape(Ln, H) + inc_p, dt, "dpos", f32_floor=1e-5)
    for b in (bout, be, bp):
        assert (b[-64:] == 7).all()


@pytest.mark.parametrize("Ln", [37, 2300])
def test_embedding_bwd_ids_beyond_24_bits(Ln):
    """25-bit ids: beside the positions of 148 tokens they fit an entry of the in-LDS sort, beside those of 9200 they do
    not and the call goes through the sort over many workgroups."""
    say(f"[embedding] vocabulary beyond 2^24, L={Ln}")
    d, dt, B, V = dev(), "f16", 4, (1 << 24) + 100
    rng = np.random.default_rng(24)
    tok = rng.choice(np.array([5, 5 + (1 << 24), 99, V - 1], np.int32), size=(B, Ln)).astype(np.int32)
    dys = encode(rng.standard_normal((B * Ln, 1), dtype=np.float32) * 0.01, dt)
    demb, dpos = torch.zeros((V, 1), dtype=torch.float16, device=d), torch.zeros((Ln, 1), dtype=torch.float16, device=d)
    L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), torch.from_numpy(tok).to(d), PAD, 2.0, 0.1, 3, 7)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 2.0, 0.1, 3, 7, dt)
    assert_close_store(demb, inc_e, dt, "demb")
    assert_close_store(dpos, inc_p, dt, "dpos")


def _class_of(ids, part_bits=6):
    """The class by which the in-LDS sort splits ids among its workgroups."""
    return (ids ^ (ids >> part_bits) ^ (ids >> 2 * part_bits)) & ((1 << part_bits) - 1)


# one class of ids at its edges (512 entries: from the next on the id that most lanes meet is taken out; 2048 entries left to sort, as
# 2600 - 552 is: from the next on in the workspace), with a frequent id, none, or nothing else; one and two halves of tokens
@pytest.mark.parametrize("tokens", [4096, 12000])
@pytest.mark.parametrize("n,frequent", [(512, 0), (513, 0), (513, 400), (2048, 0), (2049, 0), (2600, 552), (2600, 551), (3000, 2999), (3000, 3000)])
def test_embedding_bwd_large_classes(n, frequent, tokens):
    say(f"[embedding] a class of {n} tokens, {frequent} of one id, of {tokens}")
    d, dt, H, V = dev(), "f16", 8, 40000
    rng = np.random.default_rng(n + frequent + tokens)
    every = np.arange(2, V)
    own, others = every[_class_of(every) == 5], every[_class_of(every) != 5]
    tok = np.concatenate([np.full(frequent, own[17]), rng.choice(own[18:], n - frequent), rng.choice(others[:3000], tokens - n)]).astype(np.int32)
    tok[-40:] = PAD
    tok = rng.permutation(tok).reshape(1, tokens)
    dys = encode(rng.standard_normal((tokens, H), dtype=np.float32) * 0.02, dt)
    ref = None
    for _ in range(2):                                   # bit-reproducible
        demb, dpos = torch.zeros((V, H), dtype=torch.float16, device=d), torch.zeros((tokens, H), dtype=torch.float16, device=d)
        L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), torch.from_numpy(tok).to(d), PAD, 2.0, 0.1, 3, 7)
        inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 2.0, 0.1, 3, 7, dt)
        assert_close_store(demb, inc_e, dt, "demb")
        assert_close_store(dpos, inc_p, dt, "dpos")
        assert ref is None or torch.equal(ref, demb)
        ref = demb


@pytest.mark.parametrize("tokens", [129, 256])
def test_embedding_bwd_ids_of_31_bits(tokens):
    """Ids of 31 bits beside positions of 8: the sort splits them among 128 workgroups instead of 64."""
    say(f"[embedding] 31-bit ids, {tokens} tokens")
    d, dt, V = dev(), "f16", 1 << 30
    rng = np.random.default_rng(tokens)
    ids = np.array([2, 3, 2 + (1 << 29), V - 1, V - 2, 77 + (1 << 24), 77, 64, 128], np.int32)
    tok = rng.choice(ids, size=(1, tokens)).astype(np.int32)
    dys = encode(rng.standard_normal((tokens, 1), dtype=np.float32) * 0.02, dt)
    demb, dpos = torch.zeros((V, 1), dtype=torch.float16, device=d), torch.zeros((tokens, 1), dtype=torch.float16, device=d)
    L.lsq_embedding_bwd(demb, dpos, to_torch(dys, dt, d), torch.from_numpy(tok).to(d), PAD, 2.0, 0.0, 3, 7)
    # the oracle on the same tokens with the ids numbered in their order
    small = np.searchsorted(np.sort(ids), tok).astype(np.int32) + PAD + 1
    inc_e, inc_p = oracle.embedding_bwd(dys, small, len(ids) + PAD + 1, PAD, 2.0, 0.0, 3, 7, dt)
    got = demb[torch.from_numpy(np.sort(ids).astype(np.int64)).to(d)]
    assert_close_store(got, np.asarray(inc_e).reshape(-1, 1)[PAD + 1:], dt, "demb")
    assert_close_store(dpos, inc_p, dt, "dpos")
    assert int((demb != 0).sum()) <= len(ids)


# one class at the edges of the sort by counting (1, 2 or 4 threads per entry up to 64, 128 and 256 entries; from 257 on an id is taken out and
# what is left counted or radix-sorted), with 64 classes (4096 tokens) and 128 (8200: both halves of the token walk), ids met in no order
@pytest.mark.parametrize("tokens,parts", [(4096, 64), (8200, 128)])
@pytest.mark.parametrize("n,frequent", [(1, 0), (2, 0), (15, 0), (16, 0), (17, 0), (64, 0), (65, 0), (128, 0), (129, 0), (255, 3), (256, 0), (256, 256), (257, 0),
                                        (257, 1), (257, 257), (400, 143), (400, 144), (600, 344)])
def test_embedding_bwd_class_sorted_by_counting(n, frequent, tokens, parts):
    B, H, V = 2, 16, parts * 1200
    d = dev()
    r = np.random.default_rng(n * 7 + frequent + tokens)
    bits = parts.bit_length() - 1
    mix = lambda w: (w ^ (w >> bits) ^ (w >> (2 * bits))) & (parts - 1)
    ids = np.arange(V)
    mine, others = r.permutation(ids[mix(ids) == 5]), ids[mix(ids) == 6]
    tok = np.repeat(r.choice(others, 100, replace=False), -(-tokens // 100))[:tokens].astype(np.int32)       # somewhere else
    at = r.permutation(tokens)[:n]
    tok[at[:frequent]] = mine[0]
    tok[at[frequent:]] = mine[1 + np.arange(n - frequent) % (len(mine) - 1)] if n - frequent < 300 else mine[1 + r.integers(0, len(mine) - 1, n - frequent)]
    tok = tok.reshape(B, tokens // B)
    dy = encode(r.standard_normal((tokens, H), dtype=np.float32), "f32")
    demb = torch.zeros((V, H), dtype=torch.float32, device=d)
    L.lsq_embedding_bwd(demb, None, to_torch(dy, "f32", d), torch.from_numpy(tok).to(d), V, 1.0, 0.0, 1, 0)
    want = np.zeros((V, H))
    np.add.at(want, tok.reshape(-1), np.asarray(dy, dtype=np.float64).reshape(tokens, H))
    count = np.bincount(tok.reshape(-1), minlength=V)[:, None]
    # each addition rounds once: 2^-24 of a partial sum of at most sqrt-like size; 4 sigma inputs bound a sum of k by 4 k
    assert (np.abs(demb.cpu().numpy() - want) <= 2.0 ** -24 * 4 * count * np.maximum(count - 1, 0)).all()
    again = torch.zeros_like(demb)
    L.lsq_embedding_bwd(again, None, to_torch(dy, "f32", d), torch.from_numpy(tok).to(d), V, 1.0, 0.0, 1, 0)
    assert torch.equal(again, demb)


# runs of one id at the edges of the accumulation: a unit of 4 entries, a wave of 16, a range of 64 and a view of 32 about its border, slices of 8, 4, 2 packs
# and one (2, 4, 8 and 16 borders crossed), fewer slices than borders, more ranges than one look back (64); below and beyond 16384 tokens (the two sorts);
# rows of part of a column block, of one and a bit, cut packs.  Whole numbers, p = 0.5 (factors 0 and 2): every sum is exact in fp32.
@pytest.mark.parametrize("H", [8, 40, 136, 203])
@pytest.mark.parametrize("lengths,tokens", [((1, 3, 4, 5), 1500), ((15, 16, 17, 2), 1500), ((31, 33, 63, 64, 65, 1), 2000), ((127, 129, 200, 256, 6), 2500),
                                            ((500, 560, 1100, 1200, 2), 8000), ((5000, 7, 3), 6000), ((9000, 64, 1), 17000), ((66,), 66), ((65,), 65), ((64,), 64)])
def test_embedding_bwd_runs(lengths, tokens, H):
    say(f"[embedding] runs of {lengths} in {tokens} tokens, H={H}")
    d, V = dev(), 3000
    rng = np.random.default_rng(tokens + H)
    ids = rng.permutation(np.arange(2, V))
    tok, i = np.zeros(0, np.int32), 0
    while len(tok) < tokens:
        tok = np.concatenate([tok, np.full(lengths[i % len(lengths)], ids[i], np.int32)])
        i += 1
    tok = rng.permutation(tok[:tokens]).reshape(1, tokens)
    dys = rng.integers(-8, 9, size=(tokens, H)).astype(np.float32)
    d0 = rng.integers(-8, 9, size=(V, H)).astype(np.float32)
    inc_e, inc_p = oracle.embedding_bwd(dys, tok, V, PAD, 2.0, 0.5, 3, 7, "f32")
    demb, dpos = torch.from_numpy(d0).to(d), torch.zeros((tokens, H), device=d)
    L.lsq_embedding_bwd(demb, dpos, torch.from_numpy(dys).to(d), torch.from_numpy(tok).to(d), PAD, 2.0, 0.5, 3, 7)
    assert np.array_equal(demb.cpu().numpy(), (d0 + inc_e).astype(np.float32))
    assert np.array_equal(dpos.cpu().numpy(), inc_p.astype(np.float32))
    half = torch.from_numpy(d0).to(d).half()
    L.lsq_embedding_bwd(half, None, torch.from_numpy(dys).to(d).half(), torch.from_numpy(tok).to(d), PAD, 2.0, 0.5, 3, 7)
    assert torch.equal(half, demb.half())                    # one rounding per call


# the same on both sides of the tokens from which a crossing run leaves a partial row per range: runs that fill ranges, that end with them, that start in them
@pytest.mark.parametrize("H", [8, 40, 136, 203])
@pytest.mark.parametrize("lengths,tokens", [((5000, 64, 63, 65, 1, 128, 127, 129, 20), 16385), ((5000, 64, 63, 65, 1, 128, 127, 129, 20), 16384), ((64,), 33000), ((40000,), 40000),
                                            ((3, 30000, 190, 193, 2), 65600)])
def test_embedding_bwd_runs_that_cross_ranges(lengths, tokens, H):
    test_embedding_bwd_runs(lengths, tokens, H)


def test_embedding_bwd_one_id_takes_time_in_proportion_to_the_tokens():
    """Four times the tokens of one id: four times the rows to add.  A search for the run's ends by each of its workgroups makes it 11 times, and 16 further on."""
    d, H, us = dev(), 1280, []
    for rows in (1 << 18, 1 << 20):
        say(f"[embedding] one id in {rows} tokens")
        tok = torch.full((rows // 1024, 1024), 7, dtype=torch.int32, device=d)
        dy = torch.ones((rows, H), dtype=torch.bfloat16, device=d)
        demb, dpos = torch.zeros((50, H), dtype=torch.bfloat16, device=d), torch.zeros((1024, H), dtype=torch.bfloat16, device=d)
        times = []
        for _ in range(4):
            demb.zero_()
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            L.lsq_embedding_bwd(demb, dpos, dy, tok, PAD, 1.0, 0.0, 3, 7)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        assert (demb[7] == rows).all() and demb.float().sum() == rows * H       # powers of two: exact in any order
        us.append(min(times[1:]))
    assert us[1] < 8 * us[0], us
