"""Select at the row lengths where its kernels and their keys per thread change, with and without ties."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_01068_amd import binding as fk
from paper_2502_01068_amd import workloads as wl

pytestmark = pytest.mark.gpu
W = 8


@pytest.mark.parametrize("P", [1, 256, 257, 4093, 4094, 8189, 8190, 16381, 16382, 24573, 24574, 32765, 32766, 65533])
@pytest.mark.parametrize("path", [1, 2])
def test_select_row_edges(P, path):
    print("case: select rows P=%d path %d" % (P, path), flush=True)
    ctx = fk.Context(max_total_tokens=P + W, max_seqs=1)
    ctx.fkv_set_select_path(path)
    shape = fk.make_shape(P + W)
    plain = wl.random_scores(90, 2, P)
    rows = np.concatenate([plain, np.round(plain * P) / P, np.maximum(plain - np.quantile(plain, 0.9), 0),
                           -plain[:1], np.full((1, P), 0.5, np.float32)]).astype(np.float32)
    dev = torch.from_numpy(rows).cuda()
    for k in sorted({W, min(W + 1, P + W), W + P // 16, W + P // 5, W + P - 1, W + P}):
        idx = ctx.fkv_select_topk(shape, dev, k).cpu().numpy()
        for r in range(len(rows)):
            np.testing.assert_array_equal(idx[r], oracle.select_topk(rows[r], W, k), err_msg="row %d k %d" % (r, k))
    assert ctx.fkv_query_error() == 0
    ctx.close()


@pytest.mark.parametrize("P", [300, 4093, 16381, 24573, 32765])
@pytest.mark.parametrize("values", [2, 3, 20])
def test_select_few_distinct_values(P, values):
    """More equal keys in the threshold's bin than the list holds: the interval shrinks to the values it holds."""
    print("case: select P=%d, %d distinct values" % (P, values), flush=True)
    ctx = fk.Context(max_total_tokens=P + W, max_seqs=1)
    ctx.fkv_set_select_path(1)
    gen = np.random.default_rng(P + values)
    rows = np.stack([gen.uniform(-1, 1, values).astype(np.float32)[gen.integers(0, values, P)],
                     (1 + gen.integers(0, values, P) * 2.0 ** -23).astype(np.float32)])  # neighbouring floats
    rows[0, P // 2] = 1e30  # one key far away: the others share a bin of the first pass
    for k in sorted({W + 1, W + P // 10, W + P // 2, W + P - P // 10, W + P - 1}):
        idx = ctx.fkv_select_topk(fk.make_shape(P + W), torch.from_numpy(rows).cuda(), k).cpu().numpy()
        for r in range(len(rows)):
            np.testing.assert_array_equal(idx[r], oracle.select_topk(rows[r], W, k), err_msg="row %d k %d" % (r, k))
    assert ctx.fkv_query_error() == 0
    ctx.close()


@pytest.mark.parametrize("lengths", [[24000, 1500, 8189, 8190, 9, 40], [16000] + [700, 4093, 4094] * 4, [30000, 300, 12000, 8, 5000], [8189, 8190, 1]])
def test_select_mixed_lengths(lengths):
    """Rows that take fewer keys per thread than the longest one of their launch."""
    print("case: select mixed lengths %s.. (%d)" % (lengths[:4], len(lengths)), flush=True)
    total = sum(lengths) + W * len(lengths)
    ctx = fk.Context(max_total_tokens=total, max_seqs=len(lengths))
    ctx.fkv_set_select_path(1)
    shape = fk.make_shape([P + W for P in lengths])
    rows = wl.random_scores(91, 3, sum(lengths))
    rows[1] = np.round(rows[1] * 64) / 64
    for counts in ([W + P // 9 for P in lengths], [W + P for P in lengths]):
        idx = ctx.fkv_select_topk(shape, torch.from_numpy(rows).cuda(), counts).cpu().numpy()
        for r in range(3):
            at = out = 0
            for P, k in zip(lengths, counts):
                np.testing.assert_array_equal(idx[r, out:out + k], oracle.select_topk(rows[r, at:at + P], W, k), err_msg="row %d P %d" % (r, P))
                at += P
                out += k
    assert ctx.fkv_query_error() == 0
    ctx.close()


# The last value: keys per thread of the resident kernel, 0: the launch chain (test_launches_host.py looks at the launches).
MANY_LONG_ROWS = [
    (64, [32765], 8), (64, [32766], 16), (64, [39092], 16), (64, [65533], 16), (64, [65534], 32), (40, [33000, 34000], 16), (64, [70000], 32),
    (64, [24600, 33000], 32), (64, [131069], 32), (64, [131070], 0), (64, [40000, 33000, 33000], 0),
]


@pytest.mark.parametrize("n_rows,lengths", [c[:-1] for c in MANY_LONG_ROWS])
def test_select_many_long_rows(n_rows, lengths):
    """More slices of 8192 keys than blocks are resident: larger slices, or the launch chain.  The same indices from both."""
    print("case: select %d rows of %s" % (n_rows, lengths), flush=True)
    ctx = fk.Context(max_total_tokens=sum(lengths) + W * len(lengths), max_seqs=len(lengths))
    shape = fk.make_shape([P + W for P in lengths], n_q_heads=64)
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths))
    rows = torch.rand((n_rows, sum(lengths)), device="cuda", generator=gen)
    rows[1] = (rows[1] * 64).round() / 64
    counts = [W + P // 11 for P in lengths]
    got = ctx.fkv_select_topk(shape, rows, counts).clone()
    ctx.fkv_set_select_path(1)
    assert torch.equal(got, ctx.fkv_select_topk(shape, rows, counts))
    np.testing.assert_array_equal(got[1, :counts[0]].cpu().numpy(), oracle.select_topk(rows[1, :lengths[0]].cpu().numpy(), W, counts[0]))
    assert ctx.fkv_query_error() == 0
    ctx.close()
