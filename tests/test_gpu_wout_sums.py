"""Scores and window output where the output's pass leaves the window sums (the logits of every tile kept, one exchange): at the edges
of tiles, waves and splits, against the two passes over K; and where the sums do not come, so that K is read again after all."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu
# A probability is 2^x; both forms round x (at most 32 in size here: 2^-20) twice on its way: 4 * 2^-20 * ln 2.
TOL = dict(rtol=4e-6, atol=1e-37)
# The last value: whether the first launch leaves window sums (test_launches_host.py looks at the launches of these calls).
CASES = [
    ([9], 32, 8, "avg", 7, 8, True, False), ([32], 28, 7, "avg", 7, 8, True, False), ([33], 32, 8, "max", 7, 8, True, True),
    ([257], 28, 4, "avg", 15, 8, True, True), ([2048], 32, 8, "avg", 7, 3, True, True), ([8193], 32, 8, "max", 31, 8, False, True),
    ([32767], 32, 8, "avg", 7, 8, True, True), ([32768], 28, 4, "max", 1, 5, True, True), ([32769], 32, 8, "avg", 7, 8, True, False),
    ([16384], 64, 8, "avg", 7, 8, True, True), ([16385], 64, 8, "avg", 7, 8, True, False), ([4000], 56, 8, "max", 5, 7, True, True),
    ([900], 4, 1, "avg", 7, 8, True, False), ([30000], 8, 1, "avg", 7, 8, True, False), ([256], 16, 4, "avg", 7, 8, True, False),
    ([257], 16, 4, "max", 7, 8, True, True), ([3840], 16, 2, "avg", 7, 8, True, True), ([3841], 16, 2, "avg", 7, 8, True, False),
    ([5000, 16000], 32, 8, "avg", 7, 8, True, True), ([700, 9, 1024], 32, 8, "max", 7, 8, True, True),
    ([300 + 97 * i for i in range(8)], 64, 8, "avg", 3, 8, True, True), ([3000 - i for i in range(8)], 28, 4, "avg", 7, 8, True, True),
    ([1500] * 16, 4, 1, "avg", 7, 8, True, False), ([1500, 700] * 8 + [9], 4, 1, "avg", 7, 8, True, True), ([3000] * 16, 8, 2, "max", 7, 8, True, True),
    ([8000] * 3, 8, 2, "avg", 7, 8, True, False), ([12000, 9000, 9000], 12, 3, "avg", 7, 8, True, True), ([60] * 33, 8, 2, "avg", 7, 8, True, False),
    ([1024] * 32, 32, 8, "avg", 7, 8, True, True), ([1025] + [600] * 31, 32, 8, "avg", 7, 8, True, False),
]


def _inputs(lengths, hq, hkv, window=8):
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + hq)
    q = 2.0 * torch.randn((len(lengths), window, hq, 128), device="cuda", generator=gen, dtype=torch.bfloat16)
    return (q,) + tuple(torch.randn((sum(lengths), hkv, 128), device="cuda", generator=gen, dtype=torch.bfloat16) for _ in range(2))


def _check(got, want):
    assert torch.equal(got[2], want[2])
    torch.testing.assert_close(got[0], want[0], **TOL)
    torch.testing.assert_close(got[1], want[1], **TOL)


@pytest.mark.parametrize("lengths,hq,hkv,pool,pool_kernel,window,causal,sums", CASES)
def test_matches_two_passes(lengths, hq, hkv, pool, pool_kernel, window, causal, sums):
    print("case: window sums lengths=%s.. (%d) hq=%d hkv=%d %s %d w=%d" % (lengths[:4], len(lengths), hq, hkv, pool, pool_kernel, window), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=hq, n_kv_heads=hkv, pool_mode=pool, pool_kernel=pool_kernel, window=window, causal=causal)
    q, k, v = _inputs(lengths, hq, hkv, window)
    ctx.fkv_set_score_path(1)
    want = ctx.fkv_score_window_output(shape, q, k, v)
    ctx.fkv_set_score_path(0)
    first = ctx.fkv_score_window_output(shape, q, k, v)
    _check(first, want)
    if not sums:
        assert torch.equal(first[0], want[0])
    ctx.fkv_score_window(shape, q, k)  # shares the mailboxes
    again = ctx.fkv_score_window_output(shape, q, k, v)
    assert all(torch.equal(x, y) for x, y in zip(first, again))
    assert ctx.fkv_query_error() == 0
    ctx.close()


def test_without_the_sums_k_is_read_again():
    """A wait limit of 1 us, which is less than the blocks of a long input end apart, and the error flag of another call: the scores
    come from a second pass then, which shows in their last bits, and no flag is raised."""
    print("case: window sums that do not come", flush=True)
    lengths = [32768]
    ctx = fk.Context(max_total_tokens=32768, max_seqs=1)
    shape = fk.make_shape(lengths, pool_mode="avg")
    q, k, v = _inputs(lengths, 32, 8)
    want = [t.clone() for t in ctx.fkv_score_window_output(shape, q, k, v)]

    def read_again():
        got = ctx.fkv_score_window_output(shape, q, k, v)
        _check(got, want)
        assert not torch.equal(got[0], want[0])

    ctx.fkv_set_wait_limit(1)
    for _ in range(3):
        read_again()
    assert ctx.fkv_query_error() == 0
    ctx.fkv_set_wait_limit(0)  # the mark of the blocks that gave up is gone with their call: sums again
    for _ in range(2):
        assert all(torch.equal(x, y) for x, y in zip(ctx.fkv_score_window_output(shape, q, k, v), want))
    ctx.fkv_set_wait_limit(1)
    for _ in range(3):
        ctx.fkv_score_window(shape, q, k)
    assert ctx.fkv_query_error() == 1
    read_again()
    ctx.fkv_set_wait_limit(0)
    read_again()
    ctx.fkv_clear_error()
    for _ in range(2):
        assert all(torch.equal(x, y) for x, y in zip(ctx.fkv_score_window_output(shape, q, k, v), want))
    ctx.close()


def test_replays_as_a_graph():
    print("case: window sums in a graph", flush=True)
    lengths = [3000, 7000]
    ctx = fk.Context(max_total_tokens=10000, max_seqs=2)
    shape = fk.make_shape(lengths, pool_mode="avg")
    q, k, v = _inputs(lengths, 32, 8)
    want = [t.clone() for t in ctx.fkv_score_window_output(shape, q, k, v)]
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            got = ctx.fkv_score_window_output(shape, q, k, v)
    for i in range(4):
        for t in got:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, want))
        for x, y in zip(ctx.fkv_score_window_output(shape, q, k, v), want):  # eager work between the replays
            assert torch.equal(x, y)
    ctx.close()
