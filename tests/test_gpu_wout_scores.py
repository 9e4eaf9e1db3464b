"""Scores and window output in one call where its launches differ: the row normalisers folded from one split up to several
batches of them, and the output merged beside the scores (up to 16 row tiles) or in a launch of its own.  The scores are the
two-pass kernels' up to the fp32 summation order of a row's normaliser (a few ulp of a sum of up to 70000 terms: 2e-6), the
output the stand-alone call's, bit for bit."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,Hq,Hkv,window", [
    ([70000], 4, 1, 8), ([9000], 2, 2, 3), ([8193], 4, 1, 8), ([8700], 7, 1, 8), ([20001], 64, 8, 8),
    ([3000, 2500], 32, 8, 8), ([3000, 2500, 40], 32, 8, 8), ([700] * 20 + [9] * 20, 32, 8, 8),
])
def test_scores_and_output_of_one_call(lengths, Hq, Hkv, window):
    print("case: scores + window output lengths=%s Hq=%d Hkv=%d W=%d" % (lengths[:3], Hq, Hkv, window), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + Hq)
    q = (2.0 * torch.randn((len(lengths), window, Hq, 128), device="cuda", generator=gen)).bfloat16()
    k, v = (torch.randn((sum(lengths), Hkv, 128), device="cuda", generator=gen).bfloat16() for _ in range(2))
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, window=window)
    group, tsp, out = ctx.fkv_score_window_output(shape, q, k, v)
    assert torch.equal(out, ctx.fkv_window_output(shape, q, k, v))
    ctx.fkv_set_score_path(1)
    want_group, want_tsp = ctx.fkv_score_window(shape, q, k)
    for got, want in ((group, want_group), (tsp, want_tsp)):
        assert torch.isfinite(got).all() and ((got - want).abs() <= 2e-6 * want).all()
    assert ctx.fkv_query_error() == 0
    ctx.close()
