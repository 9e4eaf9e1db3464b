"""Decode attention where its work is cut: rows that end inside a block's share, rows of one tile, tiles
with one token, more rows than blocks, and one long row next to short ones."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2502_01068_amd import binding as fk
from paper_2502_01068_amd import workloads as wl
from parity import dev_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = fk.Context(max_total_tokens=4096, max_seqs=64)
    yield c
    c.close()


@pytest.mark.parametrize("ns,Hq,Hkv", [
    ([31], 32, 8), ([33], 32, 8), ([1, 32, 1], 7, 1), ([4097], 32, 8), ([9000], 4, 1), ([20000], 8, 1),
    ([30000, 1, 65], 32, 8), ([37] * 64, 32, 8), ([5 * i + 1 for i in range(64)], 64, 8), ([640] * 33, 32, 8),
    ([390 + 3 * i for i in range(40)], 32, 8), ([2100 - i for i in range(41)], 32, 8), ([384, 385] * 4, 32, 8),
])
def test_decode_cut_rows(ctx, ns, Hq, Hkv):
    print("case: decode split n=%s.. (%d) Hq=%d Hkv=%d" % (ns[:4], len(ns), Hq, Hkv), flush=True)
    B, d, tot = len(ns), 128, sum(ns)
    q = wl.normal_bf16(70, 0, "q_win", (B, Hq, d))
    k, v = (wl.normal_bf16(70, 0, n, (tot, Hkv, d)) for n in ("k", "v"))
    shape = fk.make_shape([max(n, 8) for n in ns], n_q_heads=Hq, n_kv_heads=Hkv)
    dq, dk, dv = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    first = ctx.fkv_decode_attention(shape, dq, dk, dv, ns, "token_major")
    second = ctx.fkv_decode_attention(shape, dq, dk, dv, ns, "token_major")
    assert torch.equal(first, second)
    out, o = first.cpu().numpy().astype(np.float64), 0
    for b, n in enumerate(ns):
        if b < 4 or b == B - 1:
            ref = np.asarray(oracle.decode_attention(q[b], k[o:o + n], v[o:o + n], "token_major", None, "f64"), np.float64)
            err = np.abs(out[b] - ref) / np.abs(ref).max(axis=-1, keepdims=True)
            assert err.max() <= 1e-5, "seq %d: %.3g" % (b, err.max())
        o += n


@pytest.mark.parametrize("ns,Hkv,paged", [([64], 8, False), ([4096], 8, False), ([9000], 1, False), ([2048] * 32, 8, True)])
def test_decode_infinite_v(ctx, ns, Hkv, paged):
    """An infinite V of a token with weight > 0 gives that infinity in its column, not NaN, and nothing elsewhere."""
    print("case: decode with infinite V n=%s.. (%d) Hkv=%d paged=%s" % (ns[:4], len(ns), Hkv, paged), flush=True)
    B, d, tot, page = len(ns), 128, sum(ns), 16
    q = dev_bf16(wl.normal_bf16(71, 0, "q_win", (B, Hkv * 4, d)))
    k, v = (dev_bf16(wl.normal_bf16(71, 0, n, (tot, Hkv, d))) for n in ("k", "v"))
    shape = fk.make_shape(ns, n_q_heads=Hkv * 4, n_kv_heads=Hkv)

    def run():
        if not paged:
            return ctx.fkv_decode_attention(shape, q, k, v, ns, "token_major")
        table = torch.arange(tot // page, dtype=torch.int32, device="cuda").reshape(B, -1)
        dims = (tot // page, page, Hkv, d)
        return ctx.fkv_decode_attention_paged(shape, q, k.view(dims), v.view(dims), table, ns)

    plain = run().clone()
    vf = v.view(torch.bfloat16)
    vf[3, 0, 5], vf[ns[0] - 40, Hkv - 1, 77] = float("inf"), float("-inf")
    out = run()
    want = plain.clone().view(B, Hkv, 4, d)
    want[0, 0, :, 5], want[0, Hkv - 1, :, 77] = float("inf"), float("-inf")
    assert torch.equal(out.view(B, Hkv, 4, d), want)


@pytest.mark.parametrize("ns,Hkv", [([64], 8), ([4096], 8), ([9000], 1), ([2048] * 32, 8)])
def test_decode_without_a_finite_logit(ctx, ns, Hkv):
    """Heads whose logits are all -inf have no softmax: NaN, as 0 / 0 gives, and nothing else changes."""
    print("case: decode without a finite logit n=%s.. (%d) Hkv=%d" % (ns[:4], len(ns), Hkv), flush=True)
    B, d, tot = len(ns), 128, sum(ns)
    q = dev_bf16(wl.normal_bf16(73, 0, "q_win", (B, Hkv * 4, d))).view(torch.bfloat16)
    k, v = (dev_bf16(wl.normal_bf16(73, 0, n, (tot, Hkv, d))).view(torch.bfloat16) for n in ("k", "v"))
    shape = fk.make_shape(ns, n_q_heads=Hkv * 4, n_kv_heads=Hkv)
    q[..., 0] = -1
    want = ctx.fkv_decode_attention(shape, q, k, v, ns, "token_major").view(B, Hkv, 4, d).clone()
    k[:ns[0], 0, 0] = float("inf")
    out = ctx.fkv_decode_attention(shape, q, k, v, ns, "token_major").view(B, Hkv, 4, d)
    assert torch.isnan(out[0, 0]).all()
    want[0, 0] = out[0, 0] = 0
    assert torch.equal(out, want)


class _Layout(ctypes.Structure):  # WsLayout of csrc/fkv_api.hip
    _fields_ = [(n, ctypes.c_size_t) for n in ("partial", "rowstat", "scores_group", "scores_tsp", "counters", "fused_part", "fused_lse",
                                               "sel_long", "sel_coop", "dec_part", "dec_count", "wout_o", "wout_ms", "total")] + [("max_stat_blocks", ctypes.c_int)]


class _Ctx(ctypes.Structure):  # the first members of fkv_ctx
    _fields_ = [("device", ctypes.c_int), ("max_tokens", ctypes.c_int64), ("max_seqs", ctypes.c_int32), ("lay", _Layout), ("ws", ctypes.c_void_p)]


def test_clear_error_resets_piece_counts():
    """Counts as a cut launch leaves them (written from the host): after fkv_clear_error rows in pieces are right again."""
    print("case: decode piece counts after fkv_clear_error", flush=True)
    c = fk.Context(max_total_tokens=4096, max_seqs=2)
    q, k, v = (dev_bf16(wl.normal_bf16(72, 0, n, dims)) for n, dims in (("q_win", (2, 32, 128)), ("k", (8192, 8, 128)), ("v", (8192, 8, 128))))
    shape = fk.make_shape([8, 8])
    want = c.fkv_decode_attention(shape, q, k, v, [4096, 4096], "token_major")
    raw = _Ctx.from_address(c.handle.value)
    assert (raw.device, raw.max_tokens, raw.max_seqs) == (c.device, 4096, 2)
    assert raw.lay.dec_count + 2 * 8 * 4 <= raw.lay.wout_o < raw.lay.total
    off = (ctypes.c_uint32 * 16)(*range(1, 17))
    torch.cuda.synchronize()
    copy = fk.load().hipMemcpy  # of the runtime that the library itself uses
    copy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    assert copy(raw.ws + raw.lay.dec_count, ctypes.addressof(off), ctypes.sizeof(off), 1) == 0
    c.fkv_clear_error()
    for _ in range(2):
        out = torch.full_like(want, float("nan"))
        assert torch.equal(c.fkv_decode_attention(shape, q, k, v, [4096, 4096], "token_major", out=out), want)
    c.close()


@pytest.mark.parametrize("ns,Hkv", [([1216 + 11 * i for i in range(32)], 8), ([1248, 1249] * 32, 4), ([9000] * 9, 8), ([11000], 8)])
def test_decode_layouts_agree(ctx, ns, Hkv):
    """Both sides of 40 tiles per block, from which on a token-major cache is requested in another rhythm than a compact one:
    the same bits from both."""
    print("case: decode layouts n=%s.. (%d) Hkv=%d" % (ns[:4], len(ns), Hkv), flush=True)
    B, d, tot = len(ns), 128, sum(ns)
    gen = torch.Generator(device="cuda").manual_seed(72)
    q, k, v = (torch.randn(s, device="cuda", generator=gen).to(torch.bfloat16) for s in ((B, Hkv * 4, d), (tot, Hkv, d), (tot, Hkv, d)))
    shape = fk.make_shape(ns, n_q_heads=Hkv * 4, n_kv_heads=Hkv)
    rows = ctx.fkv_decode_attention(shape, q, k, v, ns, "token_major")
    heads = ctx.fkv_decode_attention(shape, q, k.transpose(0, 1).contiguous(), v.transpose(0, 1).contiguous(), ns, "compact")
    assert torch.equal(rows, heads)
    kf, vf = k[:ns[0]].float().double(), v[:ns[0]].float().double()
    for h in (0, Hkv * 4 - 1):
        p = torch.softmax(kf[:, h // 4] @ q[0, h].double() / d ** 0.5, 0)
        ref = p @ vf[:, h // 4]
        assert ((rows[0, h].double() - ref).abs().max() / ref.abs().max()).item() <= 1e-5
