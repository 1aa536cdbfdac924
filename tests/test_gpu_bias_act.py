"""GPU parity: fused bias + activation + dropout (FFN) through the C-ABI against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2110_05722_amd as L
from tests._util import assert_close_f32, assert_close_store, dev, say
from workloads import CONFIGS, layer_tensors, to_torch

pytestmark = pytest.mark.gpu

# (rows, ffn width, p): the FFN widths of the configurations, then buckets, ragged and generic shapes
SHAPES = [(512, 2048, 0.1), (2048, 4096, 0.1), (1024, 5120, 0.1), (1000, 768, 0.3), (37, 64, 0.0), (5, 8, 0.25),
          (3, 1536, 0.1), (7, 257, 0.2), (33, 50, 0.1), (1, 4096, 0.1),
          # hidden not a multiple of 8 (the flat walk in packs): ragged last pack, two trips, accumulators outside LDS
          (3, 13, 0.1), (4100, 1031, 0.1), (9, 8197, 0.1), (300, 5124, 0.0)]


@pytest.mark.parametrize("act", ["relu", "gelu", "gelu_tanh"])
@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("rows,hidden,p", SHAPES)
def test_bias_act_dropout_fwd_bwd(rows, hidden, p, dt, act):
    if dt == "f32" and rows * hidden > 1 << 21:
        pytest.skip("fp32 storage is exercised on the small shapes only")
    say(f"[bias_act_dropout] rows={rows} hidden={hidden} p={p} dt={dt} act={act}")
    seed, offset = 99, hidden
    t = layer_tensors(CONFIGS[0], dt, rows=rows, hidden=hidden, stream=500 + rows % 83 + hidden)
    d = dev()
    x, bias, dy = (to_torch(t[k], dt, d) for k in ("x", "bias", "dy"))
    out = L.lsq_bias_act_dropout_fwd(x, bias, act, p, seed, offset)
    ref = oracle.bias_act_dropout_fwd(t["x"], t["bias"], act, p, seed, offset, dt)
    assert_close_store(out, ref, dt, "out", f32_floor=2e-6)
    out_nb = L.lsq_bias_act_dropout_fwd(x, None, act, p, seed, offset)
    assert_close_store(out_nb, oracle.bias_act_dropout_fwd(t["x"], None, act, p, seed, offset, dt), dt, "out(no bias)",
                       f32_floor=2e-6)
    dx, dbias = L.lsq_bias_act_dropout_bwd(dy, x, bias, act, p, seed, offset)
    rdx, rdb = oracle.bias_act_dropout_bwd(t["dy"], t["x"], t["bias"], act, p, seed, offset, dt)
    assert_close_store(dx, rdx, dt, "dx", f32_floor=4e-6)
    assert_close_f32(dbias, rdb, "dbias", floor=1e-6 * np.sqrt(rows) * 4)
    # in place over dy, and without dbias
    dyc = dy.clone()
    dx2, none = L.lsq_bias_act_dropout_bwd(dyc, x, bias, act, p, seed, offset, want_dbias=False, dx=dyc)
    assert none is None and torch.equal(dx, dx2)


def test_bias_act_relu_kink_and_mask():
    say("[bias_act_dropout] ReLU at exactly zero; mask bit-exact")
    d = dev()
    x = torch.tensor([[-1.0, 0.0, 1.0, 0.0, 2.0, -0.0, 0.5, -3.0]], dtype=torch.float16, device=d)
    one = torch.ones_like(x)
    dx, _ = L.lsq_bias_act_dropout_bwd(one, x, None, "relu", 0.0, 1, 0)
    assert dx.cpu().tolist() == [[0, 0, 1, 0, 1, 0, 1, 0]]
    rows, hidden, p = 513, 520, 0.3
    ones = torch.ones((rows, hidden), dtype=torch.float16, device=d)
    out = L.lsq_bias_act_dropout_fwd(ones, None, "relu", p, 77, 5)
    keep = oracle.dropout_mask(rows * hidden, p, 77, 5).reshape(rows, hidden)
    assert np.array_equal((out != 0).cpu().numpy().astype(np.uint8), keep)


def test_bias_act_empty():
    d = dev()
    x = torch.empty((0, 64), dtype=torch.float16, device=d)
    out = L.lsq_bias_act_dropout_fwd(x, None, "gelu", 0.1, 1, 0)
    dx, dbias = L.lsq_bias_act_dropout_bwd(x, x, None, "gelu", 0.1, 1, 0)
    torch.cuda.synchronize()
    assert out.numel() == 0 and dbias.abs().sum().item() == 0


# rows that are not whole packs, in packs counted from the row's start: 63 of them per wave (the 64th lane draws for its neighbour), the cut
# pack alone in a column block, every remainder; the narrowest that is not walked flat, and the widest that is
@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("rows,hidden", [(5, 249), (9, 255), (70, 257), (33, 258), (9, 503), (9, 505), (600, 509), (2049, 511), (3, 1007), (3, 1009), (41, 1014),
                                         (17, 2013), (1, 4103), (2, 8065)])
def test_bias_act_dropout_rows_of_any_length(rows, hidden, dt):
    say(f"[bias_act_dropout] any length rows={rows} hidden={hidden} dt={dt}")
    t = layer_tensors(CONFIGS[0], dt, rows=rows, hidden=hidden, stream=900 + rows % 83 + hidden)
    d = dev()
    x, bias, dy = (to_torch(t[k], dt, d) for k in ("x", "bias", "dy"))
    for act, p in (("relu", 0.0), ("gelu", 0.3), ("gelu_tanh", 0.1)):
        out = L.lsq_bias_act_dropout_fwd(x, bias, act, p, 7, hidden)
        assert_close_store(out, oracle.bias_act_dropout_fwd(t["x"], t["bias"], act, p, 7, hidden, dt), dt, "out", f32_floor=2e-6)
        dx, dbias = L.lsq_bias_act_dropout_bwd(dy, x, bias, act, p, 7, hidden)
        rdx, rdb = oracle.bias_act_dropout_bwd(t["dy"], t["x"], t["bias"], act, p, 7, hidden, dt)
        assert_close_store(dx, rdx, dt, "dx", f32_floor=4e-6)
        assert_close_f32(dbias, rdb, "dbias", floor=1e-6 * np.sqrt(rows) * 4)
        # in place, and without the column sums or the bias
        same, _ = L.lsq_bias_act_dropout_bwd(dy.clone(), x, bias, act, p, 7, hidden, want_dbias=False)
        over = x.clone()
        L.lsq_bias_act_dropout_fwd(over, bias, act, p, 7, hidden, out=over)
        assert torch.equal(same, dx) and torch.equal(over, out)
        nb = L.lsq_bias_act_dropout_fwd(x, None, act, p, 7, hidden)
        assert_close_store(nb, oracle.bias_act_dropout_fwd(t["x"], None, act, p, 7, hidden, dt), dt, "out(no bias)", f32_floor=2e-6)


def test_one_workspace_of_the_longest_batch():
    """Feed-forward, QKV split and bias+dropout+residual backward take the workspace of 2100 rows at every smaller size."""
    say("[bias_act_dropout] one workspace for all batches")
    d = dev()
    ws = {op: torch.empty(L.lsq_workspace_bytes(op, 2100, cols), dtype=torch.uint8, device=d) for op, cols in ((1, 1281), (2, 1024), (3, 1536))}
    for rows in (1, 1057, 1600, 2048, 2049, 2100):
        x = torch.randn(rows, 1024, device=d)
        dx, db = L.lsq_bias_act_dropout_bwd(x, x, None, "relu", 0.0, 1, 0, workspace=ws[2])
        assert torch.equal(dx, x * (x > 0)) and torch.allclose(db, (x * (x > 0)).sum(0), rtol=1e-5, atol=2e-6 * rows)
        x = torch.randn(rows, 1281, device=d)
        dx, db = L.lsq_bias_dropout_residual_bwd(x, 0.0, 1, 0, workspace=ws[1])
        assert torch.equal(dx, x) and torch.allclose(db, x.sum(0), rtol=1e-5, atol=2e-6 * rows)
        g = [torch.randn(1, 8, rows, 64, device=d) for _ in range(3)]
        din, db = L.lsq_split_heads_bwd(g, 1, rows, 8, 64, workspace=ws[3])
        want = torch.stack([t[0].transpose(0, 1).reshape(rows, 512) for t in g], 1).reshape(rows, 1536)
        assert torch.equal(din, want) and torch.allclose(db, want.sum(0), rtol=1e-5, atol=2e-6 * rows)


# forward of long tensors of odd rows whose second column block is thin takes the flat walk: both sides of its lines; a row does not depend on
# the path (the first rows against a short call's, bit for bit)
@pytest.mark.parametrize("hidden,elements,dt,p", [(505, 4_000_000, "f16", 0.1), (511, 4_000_000, "bf16", 0.3), (513, 6_000_000, "f16", 0.1), (519, 6_000_000, "bf16", 0.1),
                                                  (521, 6_000_000, "f16", 0.1), (545, 30_000_000, "f16", 0.1), (553, 30_000_000, "bf16", 0.1), (505, 6_000_000, "f16", 0.0), (513, 6_000_000, "f32", 0.1)])
def test_bias_act_long_tensors_of_odd_rows(hidden, elements, dt, p):
    d = dev()
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dt]
    g = torch.Generator(device=d)
    g.manual_seed(hidden)
    bias = torch.randn(hidden, generator=g, device=d).to(tdt)
    for rows in (elements // hidden, -(-elements // hidden)):
        x = torch.randn(rows, hidden, generator=g, device=d).to(tdt)
        for act in ("relu", "gelu", "gelu_tanh"):
            say(f"[bias_act_dropout] long rows={rows} hidden={hidden} dt={dt} p={p} {act}")
            out = L.lsq_bias_act_dropout_fwd(x, bias, act, p, 5, 9)
            assert torch.equal(out[:300], L.lsq_bias_act_dropout_fwd(x[:300], bias, act, p, 5, 9))
            z = x.double() + bias.double()
            ref = z.clamp(min=0) if act == "relu" else torch.nn.functional.gelu(z, approximate="tanh" if act == "gelu_tanh" else "none")
            kept = out != 0
            # one rounding to the storage type (2^-11, 2^-8) and fp32 arithmetic: 4e-6 relative to the largest term
            err = (out.double() - ref / (1 - p)).abs()
            tol = {"f16": 2.0 ** -10, "bf16": 2.0 ** -7, "f32": 1e-5}[dt] * ref.abs() + 1e-5
            assert (err[kept] <= tol[kept]).all()
            share = ((ref.abs() > 1e-2) & ~kept).double().sum() / (ref.abs() > 1e-2).double().sum()
            assert abs(share.item() - p) < 2e-3


# rows per wave of the forward on both sides of its lines (511 workgroups of two rows in fp32, 1024 in 16 bits): a row is what a short call makes of it
@pytest.mark.parametrize("rows,hidden,dt", [(4088, 512, "f32"), (4089, 512, "f32"), (8192, 512, "bf16"), (8193, 512, "bf16"), (2044, 1281, "f32"), (2720, 1281, "f16")])
def test_bias_act_rows_per_wave(rows, hidden, dt):
    say(f"[bias_act_dropout] rows per wave rows={rows} hidden={hidden} dt={dt}")
    d = dev()
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dt]
    x, bias = torch.randn(rows, hidden, device=d).to(tdt), torch.randn(hidden, device=d).to(tdt)
    out = L.lsq_bias_act_dropout_fwd(x, bias, "gelu", 0.0, 5, 9)
    for at in (0, rows // 2 // 8 * 8, (rows - 8) // 8 * 8):
        part = slice(at, min(at + 300, rows))
        assert torch.equal(out[part], L.lsq_bias_act_dropout_fwd(x[part].clone(), bias, "gelu", 0.0, 5, 9))
