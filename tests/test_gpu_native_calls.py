"""The wrappers' native call path against the ctypes one: results must be the same, on any stream, with and without
preallocated outputs, and a valid call must have gone the way it is meant to go.  Numpy counts are not recognised by
the native path; calls without counts are refused on its behalf."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


def _flat(o):
    if isinstance(o, dict):
        return [o[k] for k in sorted(o)]
    return [t for t in (o if isinstance(o, tuple) else (o,)) if t is not None]


class _Watched:
    """The native part, with a note of what each call came back with; refuse: it recognises nothing."""

    def __init__(self, native):
        self.native, self.refuse, self.taken = native, False, []

    def __getattr__(self, name):
        def fn(*args):
            out = None if self.refuse else getattr(self.native, name)(*args)
            self.taken.append((name, out is not None))
            return out
        return fn


def test_native_and_ctypes_calls_agree(monkeypatch):
    print("case: native call path", flush=True)
    fk.load()
    watch = _Watched(fk._native)
    monkeypatch.setattr(fk, "_native", watch)
    lengths, n64 = [900, 333], lambda n: [np.int64(n)] * 2
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=2)
    shape = fk.make_shape(lengths)
    gen = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen).bfloat16()
    q, k, v, x = rnd(2, 8, 32, 128), rnd(1233, 8, 128), rnd(1233, 8, 128), rnd(1233, 256)
    qd, table = rnd(2, 32, 128), torch.arange(16, dtype=torch.int32, device="cuda").reshape(2, 8)
    heads = ctx.fkv_score_heads(shape, q, k)
    idx = ctx.fkv_select_topk(shape, heads, 40)
    idx_kv = idx[:8].contiguous()
    pages = lambda: (torch.zeros((16, 16, 8, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))

    def paged(n):
        kp, vp = pages()
        return ctx.fkv_compress_kv_paged(shape, q, k, v, n, table, kp, vp), kp, vp, ctx.fkv_decode_attention_paged(shape, qd, kp, vp, table, n)

    calls = [
        lambda n: ctx.fkv_select_topk(shape, heads, n),
        lambda n: ctx.fkv_gather_rows(shape, x, idx[0].contiguous(), n),
        lambda n: ctx.fkv_gather_kv(shape, k, v, idx_kv, n),
        lambda n: ctx.fkv_gather_kv(shape, k, None, idx_kv, n),
        lambda n: ctx.fkv_gather_kv_per_head(shape, k, v, idx, n),
        lambda n: ctx.fkv_compress_kv(shape, q, k, v, n),
        lambda n: ctx.fkv_compress_kv(shape, q, k, v, n, x=x, k_tsp_per_seq=n),
        lambda n: ctx.fkv_compress_kv(shape, q, k, v, n, x=x, k_tsp_per_seq=n, out=ctx.fkv_compress_kv(shape, q, k, v, 40, x=x, k_tsp_per_seq=40)),
        lambda n: ctx.fkv_decode_attention(shape, qd, k, v, n, "token_major"),
        paged,
    ]
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            for i, call in enumerate(calls):
                watch.taken.clear()
                a = _flat(call(40))
                assert watch.taken and all(ok for _, ok in watch.taken), watch.taken
                names = [name for name, _ in watch.taken]
                watch.taken.clear()
                b = _flat(call(n64(40)))
                # the outputs that a call reuses come from a native one
                assert [name for name, _ in watch.taken] == names and not watch.taken[-1][1], watch.taken
                torch.cuda.synchronize()
                assert len(a) == len(b) and all(s.dtype == t.dtype and torch.equal(s, t) for s, t in zip(a, b)), i
    for i, call in enumerate((lambda: ctx.fkv_score_window(shape, q, k), lambda: ctx.fkv_score_window(shape, q, k, want_tsp=False),
                              lambda: ctx.fkv_score_heads(shape, q, k), lambda: ctx.fkv_window_output(shape, q, k, v),
                              lambda: ctx.fkv_score_window_output(shape, q, k, v),
                              lambda: ctx.fkv_score_window_output(shape, q, k, v, want_tsp=False),
                              lambda: ctx.fkv_score_window(shape, q, k, *(torch.empty_like(t) for t in ctx.fkv_score_window(shape, q, k))))):
        watch.taken.clear()
        a = _flat(call())
        assert watch.taken and all(ok for _, ok in watch.taken), watch.taken
        watch.refuse = True
        b = _flat(call())
        watch.refuse = False
        assert len(a) == len(b) and all(s.dtype == t.dtype and torch.equal(s, t) for s, t in zip(a, b)), i
    sg, none = ctx.fkv_score_window(shape, q, k, want_tsp=False)
    sg2, st2 = ctx.fkv_score_window(shape, q, k)
    assert none is None and torch.equal(sg, sg2) and st2.shape == (1233 - 16,)
    sg3, st3, out = ctx.fkv_score_window_output(shape, q, k, v)
    assert torch.equal(out, ctx.fkv_window_output(shape, q, k, v)) and torch.allclose(sg3, sg2, rtol=1e-4)
    for bad in (lambda: ctx.fkv_decode_attention(shape, qd.float(), k, v, 40), lambda: ctx.fkv_select_topk(shape, heads, [40]),
                lambda: ctx.fkv_compress_kv(shape, q, k[1:], v, 40), lambda: ctx.fkv_gather_kv(shape, k.transpose(0, 1), v, idx_kv, 40)):
        with pytest.raises(ValueError):
            bad()
    with pytest.raises(fk.FkvError):
        ctx.fkv_select_topk(shape, heads, 7)
    torch.cuda.synchronize()
    assert ctx.fkv_query_error() == 0
    ctx.close()
    with pytest.raises(fk.FkvError):
        ctx.fkv_select_topk(shape, heads, 40)


def test_failed_hip_call_is_raised_once():
    """A library call that reports a failed HIP call (a stand-in here) is not made again: part of it may be enqueued."""
    print("case: native call path, failed HIP call", flush=True)
    ctx = fk.Context(max_total_tokens=300, max_seqs=1)
    shape, scores = fk.make_shape(300), torch.rand((8, 292), device="cuda")
    want = ctx.fkv_select_topk(shape, scores, 40)
    calls, lib = [], fk.load()

    @ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p)
    def failing(*_):
        calls.append(1)
        return fk.FKV_EHIP

    addresses = {name: ctypes.cast(getattr(lib, name), ctypes.c_void_p).value for name in fk.EXPORTS}
    try:
        fk._native.bind(fk.FkvShape, fk.FkvError, dict(addresses, fkv_select_topk=ctypes.cast(failing, ctypes.c_void_p).value))
        with pytest.raises(fk.FkvError, match="fkv_select_topk") as e:
            ctx.fkv_select_topk(shape, scores, 40)
        assert e.value.status == fk.FKV_EHIP and len(calls) == 1
    finally:
        fk._native.bind(fk.FkvShape, fk.FkvError, addresses)
    assert torch.equal(ctx.fkv_select_topk(shape, scores, 40), want)
    ctx.close()
