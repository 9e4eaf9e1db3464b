"""Short inputs, whose token ranges are split between two blocks: the scores of a call without the all-heads mean, which takes the
split, against those of a call with it, which does not; bit for bit.  At the edges of a range and at the most ranges and one past them.  Up to four virtual groups, which one block of four
waves takes with or without the mean, against the two-pass kernels."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


# The last value: whether the call without the mean takes blocks of four waves (test_launches_host.py looks at the launches).
CASES = [
    ([34], 32, 8, "avg", 7, 8, True), ([35, 36, 61], 32, 8, "max", 7, 8, True), ([3335], 32, 8, "avg", 7, 8, True), ([3336], 28, 4, "avg", 7, 8, True),
    ([7427], 32, 8, "max", 7, 8, True), ([7428], 32, 8, "avg", 7, 8, False), ([8192], 24, 8, "avg", 1, 7, True), ([8193], 24, 8, "max", 1, 7, False),
    ([4000], 5, 5, "avg", 15, 8, True), ([4000], 24, 6, "avg", 31, 3, True), ([900] * 7, 28, 4, "avg", 5, 8, True), ([1500, 33, 8, 4000], 28, 4, "max", 15, 8, True),
    ([1500, 33, 8, 5000], 28, 4, "max", 15, 8, False), ([2000], 16, 4, "avg", 7, 8, True), ([900] * 8, 16, 4, "max", 7, 8, True), ([300] * 8, 16, 4, "avg", 7, 8, False),
    ([20], 8, 2, "avg", 7, 8, False), ([7420], 4, 1, "avg", 7, 8, True), ([900] * 7, 56, 8, "avg", 5, 8, False),
]


@pytest.mark.parametrize("lengths,hq,hkv,pool,pool_kernel,window", [c[:-1] for c in CASES])
def test_split_ranges_give_the_same_bits(lengths, hq, hkv, pool, pool_kernel, window):
    print("case: score split lengths=%s hq=%d hkv=%d %s %d w=%d" % (lengths[:4], hq, hkv, pool, pool_kernel, window), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + hq)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=hq, n_kv_heads=hkv, pool_mode=pool, pool_kernel=pool_kernel, window=window)
    q = 2.0 * torch.randn((len(lengths), window, hq, 128), device="cuda", generator=gen, dtype=torch.bfloat16)
    k = torch.randn((sum(lengths), hkv, 128), device="cuda", generator=gen, dtype=torch.bfloat16)
    whole, mean = ctx.fkv_score_window(shape, q, k)
    split, none = ctx.fkv_score_window(shape, q, k, want_tsp=False)
    heads = ctx.fkv_score_heads(shape, q, k)
    assert none is None and torch.equal(whole.view(torch.int32), split.view(torch.int32))
    g = hq // hkv
    assert torch.allclose(heads.view(hkv, g, -1).double().mean(1), whole.double(), rtol=1e-6, atol=0)  # sums of at most 8 fp32 values
    assert torch.allclose(heads.double().mean(0), mean.double(), rtol=1e-5, atol=0)  # of at most 56
    for _ in range(3):
        assert torch.equal(ctx.fkv_score_window(shape, q, k, want_tsp=False)[0].view(torch.int32), whole.view(torch.int32))
    ctx.fkv_set_score_path(1)
    torch.testing.assert_close(split, ctx.fkv_score_window(shape, q, k)[0], rtol=2e-6, atol=1e-37)  # sums over other shares
    assert ctx.fkv_query_error() == 0
    ctx.close()


@pytest.mark.parametrize("length", [34, 2048, 6554, 12289])
def test_first_tile_without_finite_logits(length):
    """Keys of a block's first tile whose logits are -inf count for nothing, as in the two-pass kernels; a NaN one takes its KV
    head's scores with it and no other's."""
    print("case: score first tile length=%d" % length, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(length)
    ctx = fk.Context(max_total_tokens=length, max_seqs=1)
    shape = fk.make_shape([length], pool_mode="avg")
    q = 2.0 * torch.randn((1, 8, 32, 128), device="cuda", generator=gen, dtype=torch.bfloat16)
    k = torch.randn((length, 8, 128), device="cuda", generator=gen, dtype=torch.bfloat16)
    q[..., 0] = -1
    plain = ctx.fkv_score_window(shape, q, k)[0].clone()
    k[3, 2, 0] = float("inf")
    got = ctx.fkv_score_window(shape, q, k)[0].clone()
    short = ctx.fkv_score_window(shape, q, k, want_tsp=False)[0]
    assert torch.equal(got, short)
    ctx.fkv_set_score_path(1)
    torch.testing.assert_close(got, ctx.fkv_score_window(shape, q, k)[0], rtol=2e-6, atol=1e-37)  # sums over other shares, as for finite inputs
    ctx.fkv_set_score_path(0)
    k[3, 2, 0] = float("nan")
    bad = ctx.fkv_score_window(shape, q, k)[0]
    assert torch.isnan(bad[2]).all()
    others = [g for g in range(8) if g != 2]
    assert torch.equal(bad[others], plain[others]) and torch.equal(got[others], plain[others])
    ctx.close()
