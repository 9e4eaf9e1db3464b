"""Which launches the calls make, and what the context does when one of them fails (no GPU; see launches.py)."""
import pytest

import launches
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
