"""Scores of the single-pass kernel, bit for bit, against checksums recorded on gfx950.  The threshold of a selection lies
between nearly equal scores, so an ulp in a softmax row's normaliser or in a window sum can keep another token: a change
of the arithmetic has to be meant."""
import zlib

import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu

CASES = [
    ([300], 32, 8, "avg", 7, 8, 0xb449c791), ([2048], 28, 4, "max", 7, 8, 0x6a7ecf37), ([4001], 32, 8, "avg", 7, 3, 0x067be52a),
    ([12289], 32, 8, "max", 7, 8, 0x301031c9), ([20001], 32, 8, "avg", 1, 1, 0x08c7f96e), ([32768], 16, 2, "avg", 15, 8, 0x342551ed),
    ([60000], 32, 8, "max", 7, 8, 0x332aa641), ([1500, 33, 7000], 32, 8, "avg", 7, 8, 0x00204ff6),
]


def _values(n, salt):
    """n multiples of 1/64 in [-2, 2), the same on every machine."""
    x = (torch.arange(n, device="cuda", dtype=torch.int64) + salt * 1000003) * 2654435761
    x = (x ^ (x >> 15)) * 2246822519
    return (((x >> 13) & 255) - 128).to(torch.float32).div_(64).bfloat16()


def checksum(lengths, Hq, Hkv, pool, pool_kernel, window):
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=Hq, n_kv_heads=Hkv, pool_mode=pool, pool_kernel=pool_kernel, window=window)
    q = _values(len(lengths) * window * Hq * 128, 1).view(len(lengths), window, Hq, 128)
    k = _values(sum(lengths) * Hkv * 128, 2).view(sum(lengths), Hkv, 128)
    heads = ctx.fkv_score_heads(shape, q, k).cpu()
    assert ctx.fkv_query_error() == 0
    ctx.close()
    return zlib.crc32(heads.numpy().tobytes())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[0][:3])))
def test_scores_keep_their_bits(case):
    print("case: score bits %s" % (case,), flush=True)
    assert checksum(*case[:-1]) == case[-1]
