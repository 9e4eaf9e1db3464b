"""Two-pass score kernels where the blocks' shares of tokens end: sequences that do not divide evenly, last
blocks of a few tokens, more than one wave of blocks, and wide groups that share one K tile."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_01068_amd import binding as fk
from paper_2502_01068_amd import workloads as wl
from parity import assert_scores_close, dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,Hq,Hkv,pool_kernel", [
    ([1000, 37, 9], 32, 8, 7), ([8 + 123], 32, 8, 7), ([31400], 32, 8, 15), ([5003, 4999, 8], 64, 8, 7),
    ([300] * 40, 32, 8, 1), ([2049, 130], 56, 8, 31), ([4100], 28, 4, 7),
])
def test_scores_token_shares(lengths, Hq, Hkv, pool_kernel):
    print("case: score shares lengths=%s Hq=%d Hkv=%d kernel=%d" % (lengths[:3], Hq, Hkv, pool_kernel), flush=True)
    seqs = [wl.make_sequence(80 + b, L, n_q_heads=Hq, n_kv_heads=Hkv, with_x=False, with_v=False) for b, L in enumerate(lengths)]
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    ctx.fkv_set_score_path(1)
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, pool_kernel=pool_kernel, pool_mode="avg")
    sg, st = ctx.fkv_score_window(shape, dev_bf16(np.stack([s["q_win"] for s in seqs])),
                                  dev_bf16(np.concatenate([s["k"] for s in seqs])))
    torch.cuda.synchronize()
    sg, st = sg.cpu().numpy(), st.cpu().numpy()
    at = 0
    for b, s in enumerate(seqs):
        P = lengths[b] - 8
        if b < 3 and P:
            ref = oracle.score_window(s["q_win"], s["k"], pool_kernel, "avg", precision="f32")
            assert_scores_close(sg[:, at:at + P], ref["scores_group"], "group seq %d" % b)
            assert_scores_close(st[at:at + P], ref["scores_tsp"], "tsp seq %d" % b)
        at += P
    ctx.close()
