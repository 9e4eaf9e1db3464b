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
