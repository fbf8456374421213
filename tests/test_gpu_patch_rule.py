"""Which weighted graphs are searched patch by patch: the rule's edges, each
with every output against the oracle (integers, and quotients of the same
integers, so all must be identical)."""
import numpy as np
import pytest

import graphgen
import oracle
import paper_1409_0035_amd as cc

pytestmark = pytest.mark.gpu
OUT = ("S_hyb", "S_samp", "S_piv", "S_pub", "pivot", "delta", "sampsum", "src_sum", "samples", "dmat", "D")


def _check(g, k, search):
    rg = graphgen.transpose(g) if g.directed else None
    samples = np.asarray(oracle.draw_samples(g.n, k, 3), dtype=np.int32)
    ref = oracle.estimate_all(g, samples, threads=8, reverse_graph=rg)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        res = cc.cc_estimate(ctx.handle, gh, k, seed=3, outputs=OUT)
        assert cc.cc_last_timing(ctx.handle)["search"] == search
        for f in OUT:
            if f in ref:
                assert np.array_equal(res[f], np.asarray(ref[f]).astype(res[f].dtype).reshape(res[f].shape)), f
        ctx.release(gh)


def _strip_with_hub(joined, directed=False):
    """A strip of 8 x 2000 nodes and one more node joined to `joined` of them,
    400 columns' worth of nodes apart or less, each in a patch of its own."""
    g = graphgen.grid(8, 2000, 4)
    deg = np.diff(g.row_ptr)
    src, dst = np.repeat(np.arange(g.n), deg), g.col_idx
    keep = src < dst
    far = (np.arange(joined) * (2000 // joined) + 3).astype(np.int64)
    s = np.concatenate([src[keep], np.full(joined, g.n)])
    d = np.concatenate([dst[keep], far])
    w = np.random.default_rng(joined).integers(1, 1000, s.size).astype(np.int32)
    g = graphgen.csr_from_arcs(g.n + 1, s, d, w)
    return graphgen.with_lengths(graphgen.symmetric_digraph(g), 1, 700, 5) if directed else g


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("joined,search", [(20, cc.CC_SEARCH_PATCHES), (50, cc.CC_SEARCH_WEIGHTED)])
def test_patch_with_many_neighbours(joined, search, directed):
    """A patch next to 31 others at most has a slot in each; past that the
    graph is searched without patches, in the caller's order."""
    _check(_strip_with_hub(joined, directed), 12, search)


def _ring(n, reach):
    i = np.repeat(np.arange(n), reach)
    j = (i + np.tile(np.arange(1, reach + 1), n)) % n
    return graphgen.csr_from_arcs(n, i, j, np.random.default_rng(reach).integers(1, 1000, i.size).astype(np.int32))


def _grid_with_extras(every):
    """A grid of eight neighbours, every so-many-th node also joined to the next but one: two arcs without a slot."""
    g = graphgen.grid(30, 40, 8)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    keep = src < g.col_idx
    v = np.arange(0, g.n - 2, every)
    v = v[v % 40 < 38]
    s, d = np.concatenate([src[keep], v]), np.concatenate([g.col_idx[keep], v + 2])
    return graphgen.csr_from_arcs(g.n, s, d, np.random.default_rng(every).integers(1, 1000, s.size).astype(np.int32))


def _grid_with_wide_lengths(share):
    """Lengths of 2^24 and more find no slot."""
    g = graphgen.grid(16, 32, 8)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    keep = src < g.col_idx
    r = np.random.default_rng(7)
    w = np.where(r.random(int(keep.sum())) < share, 1 << 24, r.integers(1 << 20, 1 << 21, int(keep.sum())))
    return graphgen.csr_from_arcs(g.n, src[keep], g.col_idx[keep], w.astype(np.int32))


def _grid_then_random():
    """64 patches of a grid first, which look well, then as many arcs between random nodes."""
    g = graphgen.grid(128, 128, 4)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    keep = src < g.col_idx
    r = np.random.default_rng(9)
    m = 20_000
    tail = g.n + np.arange(m)
    s = np.concatenate([src[keep], tail, g.n + r.integers(0, m, 2 * m)])
    d = np.concatenate([g.col_idx[keep], np.concatenate([[g.n - 1], tail[:-1]]), g.n + r.integers(0, m, 2 * m)])
    return graphgen.csr_from_arcs(g.n + m, s, d, r.integers(1, 1000, s.size).astype(np.int32))


RULE = {
    "ring-4-all-in-slots": (lambda: _ring(1500, 4), cc.CC_SEARCH_PATCHES),
    "ring-5-a-fifth-without": (lambda: _ring(1500, 5), cc.CC_SEARCH_WEIGHTED),
    "ring-6-a-third-without": (lambda: _ring(1500, 6), cc.CC_SEARCH_WEIGHTED),
    "grid-a-few-without": (lambda: _grid_with_extras(5), cc.CC_SEARCH_PATCHES),
    "grid-an-eighth-without": (lambda: _grid_with_extras(1), cc.CC_SEARCH_WEIGHTED),
    "wide-lengths-a-few": (lambda: _grid_with_wide_lengths(0.05), cc.CC_SEARCH_PATCHES),
    "wide-lengths-a-fifth": (lambda: _grid_with_wide_lengths(0.2), cc.CC_SEARCH_WEIGHTED),
    "grid-then-random": (_grid_then_random, cc.CC_SEARCH_WEIGHTED),
}


@pytest.mark.parametrize("name", list(RULE))
def test_arcs_without_a_slot(name):
    """Arcs that lie inside a patch and find no slot there, up to a tenth of all
    arcs; past that, and where later patches are not local, k_wsearch."""
    make, search = RULE[name]
    g = make()
    _check(g, 9 if g.n > 5000 else 33, search)


def test_rounds_that_run_out_belong_to_the_setting():
    """A bucket width of 1 lets a front over 1,000 x 1,000 nodes advance so little
    that the rounds run out; the next estimate at the default width goes by
    patches again, and both agree."""
    g = graphgen.grid(1000, 1000, 8, 0.1, 1, 100_000, seed=1)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        width = cc.cc_graph_get_tuning(gh)["delta"]
        got = []
        for delta, search in ((1, cc.CC_SEARCH_WEIGHTED), (width, cc.CC_SEARCH_PATCHES)):
            cc.cc_graph_set_tuning(gh, delta=delta)
            got.append(cc.cc_estimate(ctx.handle, gh, 1, seed=1, outputs=("delta", "src_sum")))
            t = cc.cc_last_timing(ctx.handle)
            print(f"  width {delta}: search {t['search']}, {t['levels']} rounds, {t['total_ms']:.1f} ms", flush=True)
            assert t["search"] == search
        assert np.array_equal(got[0]["delta"], got[1]["delta"]) and got[0]["src_sum"][0] == got[1]["src_sum"][0]
        ctx.release(gh)


@pytest.mark.parametrize("k", [7, 39, 40, 79, 81, 159, 161, 321, 512, 513])
def test_groups_of_samples(k):
    """Few patches: samples in 8, 16, 32 or 64 groups (more from 40, 80, 160 samples
    on, four a group at least), the last samples of a group missing."""
    _check(graphgen.grid(20, 33, 8, 0.1, 1, 1000, seed=5), k, cc.CC_SEARCH_PATCHES)


def test_first_look_after_a_change_of_step():
    """The rounds that a search enqueues before its first look are those of the
    last search at the same bucket width: after one at width 1, which runs
    thousands, an estimate at the default width enqueues its own few."""
    g = graphgen.grid(300, 300, 8, 0.1, 1, 1_000_000, seed=2)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        width = cc.cc_graph_get_tuning(gh)["delta"]
        seen = []
        for delta in (width, 1, width, width):
            cc.cc_graph_set_tuning(gh, delta=delta)
            cc.cc_estimate(ctx.handle, gh, 2, seed=1, outputs=("delta",))
            t = cc.cc_last_timing(ctx.handle)
            assert t["search"] == cc.CC_SEARCH_PATCHES
            seen.append((t["levels"], t["launches"]))
        print(f"  rounds and launches {seen}")
        assert seen[1][0] > 10 * seen[0][0]
        # looks come after 16 rounds and half as many again each time, then once after the rounds of the last call
        assert seen[2][1] <= 2 * seen[2][0] + 40 and seen[3][1] <= seen[3][0] + 40
        ctx.release(gh)
