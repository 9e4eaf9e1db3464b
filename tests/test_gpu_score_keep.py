"""Score kernel that keeps part of the logits and reads the rest of K again (longer inputs, wide groups): block
shares around its tile counts, against the two-pass kernels everywhere and the oracle on some rows; its
failure path, forced from the host by a wait limit of 1 us."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_01068_amd import binding as fk
from paper_2502_01068_amd import workloads as wl
from parity import assert_scores_close, dev_bf16

pytestmark = pytest.mark.gpu


def _inputs(lengths, Hq, Hkv):
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + Hq)
    q = torch.randn((len(lengths), 8, Hq, 128), device="cuda", generator=gen).bfloat16()
    return q, torch.randn((sum(lengths), Hkv, 128), device="cuda", generator=gen).bfloat16()


@pytest.mark.parametrize("lengths,Hq,Hkv,pool_mode,pool_kernel", [
    ([64001], 32, 8, "max", 7), ([137000], 32, 8, "avg", 7), ([20000, 31000, 9, 40000], 32, 8, "avg", 15), ([131072], 28, 4, "max", 1),
    ([9], 64, 8, "avg", 7), ([2056], 64, 8, "max", 7), ([16001, 8], 64, 8, "avg", 7), ([40000], 56, 8, "max", 31), ([72000], 64, 8, "avg", 7),
    ([700] * 60, 64, 8, "avg", 7), ([72000], 32, 8, "avg", 7), ([80000, 8000], 32, 8, "max", 5), ([22000], 64, 8, "avg", 7),
])
def test_matches_two_pass(lengths, Hq, Hkv, pool_mode, pool_kernel):
    print("case: score keep lengths=%s Hq=%d Hkv=%d %s %d" % (lengths[:4], Hq, Hkv, pool_mode, pool_kernel), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, pool_mode=pool_mode, pool_kernel=pool_kernel)
    q, k = _inputs(lengths, Hq, Hkv)
    ctx.fkv_profile_enable(True)
    got = ctx.fkv_score_window(shape, q, k)
    heads = ctx.fkv_score_heads(shape, q, k)
    launches = ctx.fkv_profile_read()
    assert launches["k_score_fused"][1] == 2 and launches["k_stats"][1] == 0   # resident launches, not the two-pass kernels
    ctx.fkv_profile_enable(False)
    again = ctx.fkv_score_window(shape, q, k)
    assert all(torch.equal(x, y) for x, y in zip(got, again))
    ctx.fkv_set_score_path(1)
    for x, y in zip(got + (heads,), ctx.fkv_score_window(shape, q, k) + (ctx.fkv_score_heads(shape, q, k),)):
        torch.testing.assert_close(x, y, rtol=2e-6, atol=1e-37)
    L = lengths[0]
    if L <= 20000:
        bits = lambda t: t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
        ref = oracle.score_window(bits(q[0]), bits(k[:L]), pool_kernel, pool_mode, precision="f32")
        assert_scores_close(got[0][:, :L - 8].cpu().numpy(), ref["scores_group"], "group")
    assert ctx.fkv_query_error() == 0
    ctx.close()


def test_wait_limit_fails_loudly_and_recovers():
    print("case: score keep wait limit", flush=True)
    lengths = [9000]
    ctx = fk.Context(max_total_tokens=9000, max_seqs=1)
    shape = fk.make_shape(lengths, n_q_heads=64)
    q, k = _inputs(lengths, 64, 8)
    want = [t.clone() for t in ctx.fkv_score_window(shape, q, k)]
    ctx.fkv_set_wait_limit(1)
    for _ in range(3):
        bad = ctx.fkv_score_window(shape, q, k)
    assert ctx.fkv_query_error() == 1
    assert all(torch.isnan(t).all() for t in bad)
    ctx.fkv_clear_error()
    ctx.fkv_set_wait_limit(0)
    for _ in range(2):
        assert all(torch.equal(x, y) for x, y in zip(ctx.fkv_score_window(shape, q, k), want))
    assert ctx.fkv_query_error() == 0
    ctx.close()
