"""Row gathers where a block's chunks lie in one sequence or in several, at the edges of its chunks and of the eight prefix sums a
step of the sequence search takes: copies, so bit for bit."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


def _indices(gen, lengths, counts, rows):
    return torch.cat([torch.stack([torch.randperm(n, device="cuda", generator=gen)[:c].sort().values for _ in range(rows)])
                      for n, c in zip(lengths, counts)], dim=1).to(torch.int32).contiguous()


@pytest.mark.parametrize("lengths,counts", [
    ([40], [9]), ([5000], [513]), ([40] * 8, [8] * 8), ([40] * 9, [8, 40, 8, 9, 8, 33, 8, 8, 8]), ([50 + i for i in range(64)], [8 + i % 5 for i in range(64)]),
    ([3000, 9, 700], [1025, 8, 300]),
])
@pytest.mark.parametrize("row_elems", [8, 24, 128, 4096])
def test_gathered_rows(lengths, counts, row_elems):
    print("case: gather rows lengths=%s.. (%d) row=%d" % (lengths[:3], len(lengths), 2 * row_elems), flush=True)
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + row_elems)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=32, n_kv_heads=8)
    base = [sum(lengths[:b]) for b in range(len(lengths))]
    first = torch.repeat_interleave(torch.tensor(base, device="cuda"), torch.tensor(counts, device="cuda"))
    x = torch.randint(-2**15, 2**15, (sum(lengths), row_elems), device="cuda", dtype=torch.int16, generator=gen).view(torch.bfloat16)
    idx = _indices(gen, lengths, counts, 1)
    got = ctx.fkv_gather_rows(shape, x, idx[0], counts)
    assert torch.equal(got.view(torch.int16), x[first + idx[0]].view(torch.int16))
    if row_elems != 128:
        ctx.close()
        return
    kv = torch.randint(-2**15, 2**15, (2, sum(lengths), 8, 128), device="cuda", dtype=torch.int16, generator=gen).view(torch.bfloat16)
    idx = _indices(gen, lengths, counts, 8)
    want = [torch.stack([c[first + idx[g], g] for g in range(8)]) for c in kv]
    for got, w in zip(ctx.fkv_gather_kv(shape, kv[0], kv[1], idx, counts), want):
        assert torch.equal(got.view(torch.int16), w.view(torch.int16))
    page, need = 4, [-(-c // 4) for c in counts]
    table = torch.full((len(counts), max(need)), -1, dtype=torch.int32, device="cuda")
    order, at = torch.randperm(sum(need) + 3, device="cuda", generator=gen).to(torch.int32), 0
    for b, n in enumerate(need):
        table[b, :n] = order[at:at + n]
        at += n
    pools = [torch.zeros((sum(need) + 3, page, 8, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    ctx.fkv_gather_kv_paged(shape, kv[0], kv[1], idx, counts, table, pools[0], pools[1])
    o = 0
    for b, c in enumerate(counts):
        j = torch.arange(c, device="cuda")
        for pool, w in zip(pools, want):
            assert torch.equal(pool[table[b, j // page].long(), j % page].transpose(0, 1).contiguous().view(torch.int16), w[:, o:o + c].contiguous().view(torch.int16))
        o += c
    ctx.close()
