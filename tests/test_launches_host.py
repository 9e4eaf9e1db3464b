"""Which launches the calls make, and what the context does when one of them fails (no GPU; see launches.py)."""
import pytest

import launches
import test_gpu_score_split
import test_gpu_select_gather
import test_gpu_select_rows
import test_gpu_wout_sums

EHIP, EUNSUPPORTED = -6, -4


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("recorder")
    return lambda *steps: launches.run([["create", {}]] + [list(s) for s in steps], tmp)[1:]


def test_posted_mailboxes_are_not_read_after_a_failed_launch(calls):
    """The window output's first launch posts into the score mailboxes, its second one empties them.  If that one fails, no kernel
    that reads mailboxes may run before fkv_clear_error; the scores come from the two-pass kernels."""
    window, score = ("window_output", {"lengths": [8192]}), ("score", {"lengths": [8192]})
    got = calls(window, score, ("window_output", {"lengths": [8192], "refuse_launch": 1}), score, window,
                ("compress", {"lengths": [8192], "budgets": [512], "k_tsp": [1638]}), ("set", {"what": "set_score_path", "value": 2}), score,
                ("set", {"what": "set_score_path", "value": 0}), ("clear_error", {}), window, score)
    before, failed, after = got[:2], got[2], got[3:6]
    assert [launches.kernels(r)[0].split("<")[0] for r in before] == ["k_wout_partial", "k_score_fused"]
    assert launches.kernels(before[0])[0] == "k_wout_partial<true, true>"
    assert failed["value"] == EHIP and launches.kernels(failed) == ["k_wout_partial<true, true>"]
    for r in after:
        assert r["value"] == 0 and all(l["wait_ticks"] == 0 for l in r["launches"]), r
    assert launches.kernels(after[0])[0].startswith("k_stats") and launches.kernels(after[2])[0].startswith("k_stats")
    assert launches.kernels(after[1])[0] == "k_wout_partial<true, false>"
    assert got[7]["value"] == EUNSUPPORTED  # the single-pass kernel and no other was asked for
    assert [launches.kernels(r) for r in got[-2:]] == [launches.kernels(r) for r in before]


def test_a_failed_first_launch_leaves_the_mailboxes_usable(calls):
    got = calls(("window_output", {"lengths": [8192], "refuse_launch": 0}), ("score", {"lengths": [8192]}))
    assert got[0]["value"] == EHIP and launches.kernels(got[1])[0].startswith("k_score_fused")


def test_window_sums_wait_no_longer_than_reading_k_again_is_worth(calls):
    """A block of the window sums that misses another block's words is as well off reading K again: 0.1 ms at most, whatever the
    context's limit; a shorter limit holds."""
    window, limit = ("window_output", {"lengths": [8192]}), lambda us: ("set", {"what": "set_wait_limit", "value": us})
    got = calls(window, limit(1000000), window, limit(5), window, limit(0), window)
    ticks = [r["launches"][0]["wait_ticks"] for r in got if r["launches"]]
    assert ticks == [10000, 10000, 500, 10000]  # of 10 ns


def test_window_sums_where_they_are_faster(calls):
    cases = test_gpu_wout_sums.CASES
    got = calls(*[("window_output", {"lengths": c[0], "hq": c[1], "hkv": c[2], "pool_kernel": c[4], "window": c[5]}) for c in cases])
    for c, r in zip(cases, got):
        assert r["value"] == 0 and launches.kernels(r)[0] == ("k_wout_partial<true, true>" if c[-1] else "k_wout_partial<true, false>"), c


def test_no_window_sums_beside_another_context(calls):
    got = calls(("window_output", {"lengths": [8192]}), ("create", {}), ("window_output", {"lengths": [8192]}), ("destroy", {}), ("window_output", {"lengths": [8192]}))
    assert [launches.kernels(r)[0] for r in got if r["launches"]] == ["k_wout_partial<true, %s>" % s for s in ("true", "false", "true")]


@pytest.mark.parametrize("paged", [False, True])
def test_every_parity_case_of_the_one_launch_takes_it(calls, paged):
    """And makes two launches of select and gather while launches are timed, which is what that test compares with."""
    cases = [(c, p) for c in test_gpu_select_gather.CASES for p in test_gpu_select_gather.POOLS[:1]]
    steps = [("compress", {"lengths": c[0], "budgets": c[1], "k_tsp": None if paged else c[2], "hidden": c[3], "hq": c[4],
                           "hkv": test_gpu_select_gather.hkv_of(c[4]), "pool_kernel": p[1], "paged": paged}) for c, p in cases]
    got = calls(*steps, ("set", {"what": "profile_enable", "value": 1}), *steps)
    for (c, _), one, two in zip(cases, got, got[len(steps) + 1:]):
        assert launches.kernels(one)[-1].startswith("k_select_gather<"), c
        assert [k.split("<")[0] for k in launches.kernels(two)[-2:]] == ["k_select", "k_gather_paged" if paged else "k_gather"], c


def _compress(n, length, budget, **kw):
    return "compress", dict({"lengths": [length] * n, "budgets": [budget] * n}, **kw)


def test_one_launch_where_it_is_faster(calls):
    """Rows and bytes of a block on both sides of the rule's lines: long rows, a share of 192 KB, 120 KB for pages from short inputs, for
    a last round of few blocks and for many rows beside hidden rows."""
    steps = [(_compress(1, 24581, 2048), True), (_compress(1, 24582, 2048), False), (_compress(1, 12000, 12000), True), (_compress(1, 24500, 24500), False),
             (_compress(1, 8192, 7500, paged=True), True), (_compress(1, 8192, 8192, paged=True), False), (_compress(1, 13000, 9000, paged=True), True),
             (_compress(48, 2400, 240), True), (_compress(33, 3000, 300), False), (_compress(32, 3000, 300), True),
             (_compress(18, 900, 90, k_tsp=[90] * 18), True), (_compress(18, 900, 90, k_tsp=[135] * 18), False), (_compress(8, 900, 90, k_tsp=[135] * 8), True)]
    got = calls(*[s for s, _ in steps])
    for (s, one), r in zip(steps, got):
        assert r["value"] == 0 and launches.kernels(r)[-1].startswith("k_select_gather<") == one, s


def test_one_launch_not_while_several_blocks_share_a_row(calls):
    got = calls(("set", {"what": "set_select_path", "value": 2}), _compress(1, 2048, 256), ("set", {"what": "set_select_path", "value": 1}), _compress(1, 2048, 256))
    assert [launches.kernels(r)[-1].split("<")[0] for r in got if r["launches"]] == ["k_gather", "k_select_gather"]


def test_ranges_split_between_blocks(calls):
    """Without the mean over all heads; with it only where a block still sees every head, or the select adds the groups' sums up."""
    cases = test_gpu_score_split.CASES
    step = lambda c, mean: ("score", {"lengths": c[0], "hq": c[1], "hkv": c[2], "pool_kernel": c[4], "window": c[5], "mean": mean})
    got = calls(*[step(c, mean) for c in cases for mean in (False, True)])
    for c, split, mean in zip(cases, got[::2], got[1::2]):
        groups = c[2] * (2 if c[1] // c[2] > 4 else 1)
        assert (launches.kernels(split) == ["k_score_fused<2, 4>"]) == c[-1], c
        assert (launches.kernels(mean) == ["k_score_fused<2, 4>"]) == (c[-1] and groups <= 4), c
        if c[-1]:
            assert split["launches"][0]["threads"] == 256 and split["launches"][0]["blocks"] <= 256


def test_slices_of_many_long_rows(calls):
    cases = test_gpu_select_rows.MANY_LONG_ROWS
    got = calls(*[("select", {"lengths": [P + 8 for P in lengths], "rows": n, "counts": [8 + P // 11 for P in lengths], "hq": 64}) for n, lengths, _ in cases])
    for c, r in zip(cases, got):
        name = launches.kernels(r)[0]
        assert r["value"] == 0 and name.startswith("k_select_coop<%d," % c[2] if c[2] else "k_sel_long_prep"), (c, name)


def test_workspace_holds_the_window_sums_of_its_tokens(calls):
    """Up to 64 heads of 4 bytes a token, 8 MB at most: a context for short inputs does not pay for long ones."""
    small, full, more = [r["value"] for r in calls(*[("workspace_bytes", {"tokens": n, "seqs": 1}) for n in (2048, 32768, 63488)])]
    assert (full - small) - (more - full) == (8 << 20) - 2048 * 256  # what grows with the tokens is linear otherwise
