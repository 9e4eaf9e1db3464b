"""Select and gather in one launch against the two launches that a timed context makes of the same call: indices and copies, so
bit for bit.  Rows at the edges of the keys per thread, parts of a row at the edges of a step, one and several sequences, rows of
8 keys per thread next to longer ones, hidden rows of any multiple of 16 bytes, everything kept and only the window kept, pages; and
rows of all heads that the select adds up from the groups' sums (ranges split between blocks), at the most ranges and one past them."""
import pytest
import torch

from paper_2502_01068_amd import binding as fk

pytestmark = pytest.mark.gpu


CASES = [
    ([4101], [64], [512], 4096, 32), ([4102], [8], [8], 24, 32), ([9], [9], [8], 8, 32), ([8], [8], [8], 8, 32), ([8197], [2048], None, 0, 32),
    ([8198], [65], [700], 136, 64), ([12293], [1229], [1230], 1024, 28), ([12294], [129], None, 0, 32), ([16389], [1000], [1639], 4096, 32),
    ([16390], [11000], None, 0, 32), ([20486], [300], [20486], 8, 64), ([24581], [2000], [2400], 4096, 32), ([24580], [2000], [24], 64, 32),
    ([23000, 2000, 8, 9, 4500], [100, 2000, 8, 8, 450], [2300, 17, 8, 9, 1111], 512, 32), ([1500 + 7 * i for i in range(64)], [130] * 64, [31] * 64, 56, 32),
    ([3000] * 9, [8, 64, 128, 63, 129, 3000, 8, 9, 257], None, 0, 28), ([3335], [300], [600], 64, 24), ([3336], [200], [301], 64, 28),
    ([7431, 9], [300, 8], [1000, 9], 64, 16), ([7440], [300], [1000], 64, 20), ([700, 2049, 8, 1300], [100] * 2 + [8, 100], [70, 205, 8, 130], 64, 32),
    ([300 + i for i in range(10)], [30] * 10, [40] * 10, 24, 32), ([300] * 8 + [77], [65, 8] * 4 + [9], None, 0, 28), ([7000], [7000], [7000], 64, 32),
]
POOLS = [("avg", 7), ("max", 1), ("avg", 15)]  # the others where the select adds up group sums: the pooling does not matter behind blocks that have all heads


def hkv_of(hq):
    return {28: 4, 20: 4, 16: 2}.get(hq, 8)


def _randn(gen, *shape):
    return torch.randn(shape, device="cuda", generator=gen, dtype=torch.bfloat16)


@pytest.mark.parametrize("lengths,budgets,k_tsp,hidden,hq,pool", [c + (p,) for c in CASES for p in POOLS if p == POOLS[0] or sum(c[0]) <= 8300])
def test_one_launch_matches_two(lengths, budgets, k_tsp, hidden, hq, pool):
    print("case: select and gather lengths=%s.. (%d) tsp=%s hidden=%d hq=%d %s" % (lengths[:3], len(lengths), k_tsp and k_tsp[:3], hidden, hq, pool), flush=True)
    hkv = hkv_of(hq)
    gen = torch.Generator(device="cuda").manual_seed(sum(lengths) + hq)
    ctx = fk.Context(max_total_tokens=sum(lengths), max_seqs=len(lengths))
    shape = fk.make_shape(lengths, n_q_heads=hq, n_kv_heads=hkv, pool_mode=pool[0], pool_kernel=pool[1])
    q, k, v = _randn(gen, len(lengths), 8, hq, 128), _randn(gen, sum(lengths), hkv, 128), _randn(gen, sum(lengths), hkv, 128)
    x = _randn(gen, sum(lengths), hidden) if k_tsp else None

    def compress():
        out = ctx.fkv_compress_kv(shape, q, k, v, budgets, x=x, k_tsp_per_seq=k_tsp)
        return {n: t.clone() for n, t in out.items() if t is not None}

    page, need = 4, [-(-c // 4) for c in budgets]
    table = torch.full((len(budgets), max(need)), -1, dtype=torch.int32, device="cuda")
    order, at = torch.randperm(sum(need) + 3, device="cuda", generator=gen).to(torch.int32), 0
    for b, n in enumerate(need):
        table[b, :n] = order[at:at + n]
        at += n
    table[0, 0] = sum(need) + 3  # outside the pool: nothing is written

    def paged():
        pools = [torch.full((sum(need) + 3, page, hkv, 128), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        return [ctx.fkv_compress_kv_paged(shape, q, k, v, budgets, table, pools[0], pools[1])] + pools

    one, one_paged = compress(), paged()
    ctx.fkv_profile_enable(True)
    ctx.fkv_profile_read()
    two, two_paged = compress(), paged()
    launches = ctx.fkv_profile_read()
    ctx.fkv_profile_enable(False)
    assert launches["k_select"][1] == 2 and launches["k_gather"][1] == 2, launches
    assert one.keys() == two.keys()
    for name in one:
        assert torch.equal(one[name].view(torch.int16), two[name].view(torch.int16)), name
    for a, b in zip(one_paged, two_paged):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    ctx.close()


def test_failed_scores_mark_every_index_and_copy_nothing():
    ctx = fk.Context(max_total_tokens=6000, max_seqs=1)
    gen = torch.Generator(device="cuda").manual_seed(3)
    shape = fk.make_shape(6000, n_q_heads=32, n_kv_heads=8)
    q, k, v, x = _randn(gen, 8, 32, 128), _randn(gen, 6000, 8, 128), _randn(gen, 6000, 8, 128), _randn(gen, 6000, 64)
    good = {n: t.clone() for n, t in ctx.fkv_compress_kv(shape, q, k, v, 500, x=x, k_tsp_per_seq=700).items()}
    out = ctx.fkv_compress_kv(shape, q, k, v, 500, x=x, k_tsp_per_seq=700)
    ctx.fkv_set_wait_limit(1)
    for n in ("k_out", "v_out", "x_out"):
        out[n].fill_(7.0)
    out = ctx.fkv_compress_kv(shape, q, k, v, 500, x=x, k_tsp_per_seq=700, out=out)
    assert ctx.fkv_query_error() != 0
    assert (out["idx_kv"] == -1).all() and (out["idx_tsp"] == -1).all()
    assert all((out[n] == 7.0).all() for n in ("k_out", "v_out", "x_out"))
    ctx.fkv_set_wait_limit(0)
    ctx.fkv_clear_error()
    again = ctx.fkv_compress_kv(shape, q, k, v, 500, x=x, k_tsp_per_seq=700)
    assert all(torch.equal(again[n].view(torch.int16), good[n].view(torch.int16)) for n in good)
    ctx.close()
