"""cc_last_timing says which search an estimate ran and whether it replayed a
captured graph: a small graph's one launch is no replay."""
import numpy as np
import pytest

import graphgen
import paper_1409_0035_amd as cc

pytestmark = pytest.mark.gpu


def _searches(ctx, gh, n, k, modes, samples):
    import torch
    out = {"S_hyb": torch.empty(n, dtype=torch.float64, device="cuda")}
    got = []
    for mode in modes:
        cc.cc_estimate_device(ctx.handle, gh, k, out, mode=mode, samples=samples)
        got.append(cc.cc_last_timing(ctx.handle)["search"])
    return got


GRAPH = cc.CC_BATCHED | cc.CC_GRAPH
CASES = {
    "small": (lambda: graphgen.ba(2000, 4, seed=1), cc.CC_SEARCH_SMALL, False),
    "past-the-small": (lambda: graphgen.ba(49153, 4, seed=1), cc.CC_SEARCH_LEVELS, True),
    "patches": (lambda: graphgen.grid(30, 40, 8, 0.1, 1, 1000, seed=1), cc.CC_SEARCH_PATCHES, True),
    "weighted": (lambda: graphgen.with_lengths(graphgen.ba(3000, 4, seed=1), 1, 50, 2), cc.CC_SEARCH_WEIGHTED, True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_search_is_named(name):
    make, search, replays = CASES[name]
    g = make()
    samples = np.arange(5, 25, dtype=np.int32)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        got = _searches(ctx, gh, g.n, 20, (cc.CC_BATCHED, GRAPH, GRAPH, cc.CC_PLAIN), samples)
        again = search | (cc.CC_SEARCH_REPLAY if replays else 0)
        assert got == [search, search, again, cc.CC_SEARCH_PLAIN]
        ctx.release(gh)


def test_small_graph_time_includes_its_error_pass():
    """total_ms runs to the last output: with the Sec. 4 outputs and the sweep
    asked for, the epilogue of a small graph counts them (they take several
    times what the estimates do)."""
    import torch
    g = graphgen.ba(20000, 4, seed=2)
    k = 256
    est = {"S_hyb": torch.empty(g.n, dtype=torch.float64, device="cuda")}
    both = {**est, **{f: torch.empty(g.n, dtype=torch.float64, device="cuda")
                      for f in ("S_err", "S_ad", "S_ad_err", "S_sweep", "S_sweep_err")}}
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        ms = []
        for out in (est, both):
            for _ in range(3):
                cc.cc_estimate_device(ctx.handle, gh, k, out, seed=1)
            t = cc.cc_last_timing(ctx.handle)
            assert t["search"] == cc.CC_SEARCH_SMALL
            assert abs(t["total_ms"] - t["traverse_ms"] - t["epilogue_ms"]) < 1e-9
            ms.append(t["epilogue_ms"])
        print(f"  epilogue {ms[0]:.4f} ms, with errors {ms[1]:.4f} ms")
        assert ms[1] > 2 * ms[0]
        ctx.release(gh)


def test_arcs_scanned_is_not_clipped():
    """A chain of 236 nodes with 2,100 parallel arcs between neighbours, and at
    its end two nodes joined by 500,000: the levels pull, and one wave reads
    the two long rows again in each of them until the search arrives, past
    2^31 / 16 arcs."""
    chain, thick, long_row = 236, 2100, 500_000
    a, b = chain, chain + 1
    i = np.arange(chain - 1)
    src = np.concatenate([np.repeat(i, thick), [chain - 1], np.full(long_row, a)])
    dst = np.concatenate([np.repeat(i + 1, thick), [a], np.full(long_row, b)])
    s, d = np.concatenate([src, dst]), np.concatenate([dst, src])
    order = np.argsort(s, kind="stable")
    n = chain + 2
    rp = np.zeros(n + 1, dtype=np.int64)
    rp[1:] = np.cumsum(np.bincount(s, minlength=n))
    assert s.size <= 1 << 21
    with cc.Context(0) as ctx:
        gh = cc.cc_graph_upload(ctx.handle, n, s.size, rp, d[order].astype(np.int32))
        res = cc.cc_estimate(ctx.handle, gh, 1, samples=[0], outputs=("src_sum",))
        t = cc.cc_last_timing(ctx.handle)
        print(f"  arcs scanned {t['arcs_scanned']}, {t['total_ms']:.1f} ms")
        assert t["search"] == cc.CC_SEARCH_SMALL and res["src_sum"][0] == n * (n - 1) // 2
        # every level from the tenth on pulls, and reads the rows of all nodes not yet found
        assert t["arcs_scanned"] > sum(2 * long_row + 2 * thick * (chain - level) for level in range(10, chain - 1))
        cc.cc_graph_release(gh)


def test_autotune_times_a_small_graphs_setting_only():
    """No knob is read by a small graph's search: the tuner keeps the setting
    and takes the time of two rounds of estimates (a warm-up and the timed
    one) instead of measuring its dozen candidates."""
    import time
    import torch
    reps = 100
    with cc.Context(0) as ctx:
        g = graphgen.ba(5000, 4, seed=1)
        gh = ctx.upload(g)
        out = {"S_hyb": torch.empty(g.n, dtype=torch.float64, device="cuda")}
        before = cc.cc_graph_get_tuning(gh)
        for _ in range(2):
            t0 = time.perf_counter()
            for _ in range(reps):
                cc.cc_estimate_device(ctx.handle, gh, 64, out, seed=1)
            one_round = time.perf_counter() - t0
        t0 = time.perf_counter()
        best, ms = cc.cc_autotune(ctx.handle, gh, 64, seed=1, reps=reps)
        took = time.perf_counter() - t0
        print(f"  {reps} estimates {one_round * 1e3:.2f} ms, the tuner {took * 1e3:.2f} ms")
        assert ms > 0 and best == before and cc.cc_graph_get_tuning(gh) == before
        assert took < 6 * one_round
        ctx.release(gh)


def test_flat_graph_is_pushed_until_pulls_end_early():
    """A random graph without hubs: at its third level some 1,600 of 49,000 nodes
    are known, so that a pull would read most of the arcs, and the search still
    pushes (their 64,000 arcs)."""
    n, deg, k = 49000, 40, 16
    r = np.random.default_rng(4)
    g = graphgen.csr_from_arcs(n, r.integers(0, n, n * deg // 2), r.integers(0, n, n * deg // 2))
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        cc.cc_estimate(ctx.handle, gh, k, seed=1, outputs=("S_hyb",))
        t = cc.cc_last_timing(ctx.handle)
        print(f"  {t['arcs_scanned'] / k / g.arcs:.3f} of {g.arcs} arcs a search")
        assert t["search"] == cc.CC_SEARCH_SMALL
        # the pushes, and pulls with more than half of the nodes known (two arcs a node and a trip's rest)
        assert t["arcs_scanned"] < k * g.arcs / 4
        ctx.release(gh)
