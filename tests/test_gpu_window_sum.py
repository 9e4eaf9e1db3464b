"""The window sum of Eq. 1, bit for bit: the score of a token is the fp32 sum of its W probabilities, each rounded by
itself.  A window row is left out by pointing its query at a sink (the last token, along a direction that nothing else
uses), so that its probability of every other token is exactly 0; the single rows' probabilities then add up to the
full call's scores in the order rows 0..3, rows 4..7, both halves."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


def _inputs(lengths, Hq, Hkv):
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + Hq)
    q = 2.0 * torch.randn((len(lengths), 8, Hq, 128), device="cuda", generator=gen)
    k = torch.randn((sum(lengths), Hkv, 128), device="cuda", generator=gen)
    q[..., 127], k[..., 127] = 0.0, 0.0
    at = 0
    for n in lengths:
        at += n
        k[at - 1, :, 127] = 64.0
    return q.bfloat16(), k.bfloat16()


@pytest.mark.parametrize("lengths,Hq,Hkv,path", [
    ([20], 32, 8, 2), ([300], 28, 4, 2), ([2049], 32, 8, 2), ([12289], 32, 8, 2), ([30000], 32, 8, 2), ([700, 33, 2000], 32, 8, 2),
    ([700, 33], 32, 8, 1), ([5000], 64, 8, 1), ([5000], 64, 8, 0), ([66000], 32, 8, 0),
])
def test_window_sum_is_the_sum_of_rounded_probabilities(lengths, Hq, Hkv, path):
    print("case: window sum lengths=%s Hq=%d Hkv=%d path=%d" % (lengths, Hq, Hkv, path), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    ctx.fkv_set_score_path(path)
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, pool_kernel=1, causal=False)
    q, k = _inputs(lengths, Hq, Hkv)
    full = ctx.fkv_score_heads(shape, q, k)
    rows = []
    for w in range(8):
        alone = torch.zeros_like(q)
        alone[..., 127] = 64.0  # logit 362 of the sink, 0 of the rest: their probability is below fp32's range
        alone[:, w] = q[:, w]
        rows.append(ctx.fkv_score_heads(shape, alone, k).cpu())
    want = (((rows[0] + rows[1]) + rows[2]) + rows[3]) + (((rows[4] + rows[5]) + rows[6]) + rows[7])
    assert (want > 0).all() and torch.equal(full.cpu(), want)
    assert ctx.fkv_query_error() == 0
    ctx.close()


@pytest.mark.parametrize("window,lengths,Hq,Hkv,path", [
    (1, [300], 32, 8, 2), (3, [2049], 32, 8, 2), (7, [12289], 28, 4, 2), (5, [40000], 32, 8, 2), (3, [700, 40], 32, 8, 1), (3, [5000], 64, 8, 0),
])
def test_infinite_key_with_a_short_window(window, lengths, Hq, Hkv, path):
    """A key whose logits are -inf in every row of the window scores 0; the matrix tile's rows past the window, whose
    queries are 0 and whose logits of that key are NaN, do not count."""
    print("case: infinite key window=%d lengths=%s Hq=%d Hkv=%d path=%d" % (window, lengths, Hq, Hkv, path), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    ctx.fkv_set_score_path(path)
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, pool_kernel=1, window=window)
    q, k = _inputs(lengths, Hq, Hkv)
    q = q[:, :window].contiguous()
    q[..., 0] = -1.0
    at = lengths[0] // 3
    k[at, :, 0] = float("inf")
    heads = ctx.fkv_score_heads(shape, q, k)
    assert torch.isfinite(heads).all()
    assert (heads[:, at] == 0).all() and (heads[:, at + 1] > 0).all()
    assert ctx.fkv_query_error() == 0
    ctx.close()
