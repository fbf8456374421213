"""Weighted graphs that can be cut into patches are searched patch by patch:
every output at the edges of that path (the smallest graphs, nodes with more
inner arcs than slots, arc lengths too large for a slot, arcs whose two
directions differ, distances near the 31-bit limit, many samples) and of the
histogram over its rows (ranges of LDS bins) against the oracle.  Distances and sums are integers, the estimates one division of exact
integers on both sides, so all must be identical."""
import sys

import numpy as np
import pytest

import graphgen
import oracle
import paper_1409_0035_amd as cc

pytestmark = pytest.mark.gpu
OUT = ("S_hyb", "S_samp", "S_piv", "S_pub", "pivot", "delta", "sampsum", "src_sum", "samples", "dmat", "D", "S_err",
       "S_ad", "S_ad_err")
LONG = ("pivot", "delta", "src_sum", "samples", "dmat", "D")  # squares of long distances leave 2^53


def _grid(rows, cols, wlo=1, whi=1000):
    return graphgen.grid(rows, cols, 8, 0.1, wlo, whi, seed=rows * cols)


def _caterpillar(spine, legs):
    """A path whose nodes carry `legs` leaves: more inner arcs than a node has slots."""
    s = np.arange(spine - 1)
    leaf = np.arange(spine, spine * (legs + 1))
    src = np.concatenate([s, (leaf - spine) // legs])
    dst = np.concatenate([s + 1, leaf])
    w = np.random.default_rng(3).integers(1, 100, src.shape[0]).astype(np.int32)
    return graphgen.csr_from_arcs(spine * (legs + 1), src, dst, w)


def _long_path(n, w):
    i = np.arange(n - 1, dtype=np.int32)
    return graphgen.csr_from_arcs(n, i, i + 1, np.full(n - 1, w, np.int32))


def _two_lengths(longest):
    """A path of 603 nodes whose length from end to end is `longest`."""
    i = np.arange(602, dtype=np.int32)
    w = np.full(602, longest // 602, np.int32)
    w[: longest % 602] += 1
    return graphgen.csr_from_arcs(603, i, i + 1, w)


def _one_way_grid():
    return graphgen.with_lengths(graphgen.symmetric_digraph(graphgen.grid(30, 41, 4)), 1, 50, 8)


CASES = {
    "grid511-general-path": (lambda: _grid(7, 73), 20),
    "grid512": (lambda: _grid(16, 32), 64),
    "grid23x61-k1": (lambda: _grid(23, 61), 1),
    "grid40x50-k9": (lambda: _grid(40, 50), 9),
    "grid30x40-k600": (lambda: _grid(30, 40), 600),
    "grid16x32-wide-lengths": (lambda: _grid(16, 32, 1 << 24, 1 << 25), 17),
    "grid25x40-unit-like": (lambda: _grid(25, 40, 1, 2), 33),
    "caterpillar-many-inner-arcs": (lambda: _caterpillar(200, 11), 40),
    "one-way-grid-round-trip": (_one_way_grid, 50),
    # the distance table one bin short of, at and past a range of LDS bins, and past the last range that is read again
    "table-36863": (lambda: _two_lengths(36862), 30),
    "table-36864": (lambda: _two_lengths(36863), 30),
    "table-36865": (lambda: _two_lengths(36864), 30),
    "table-20-ranges": (lambda: _two_lengths(20 * 36864 - 1), 9),
    "table-past-20-ranges": (lambda: _two_lengths(20 * 36864), 9),
    "path-near-the-limit": (lambda: _long_path(600, 3_580_000), 3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_patches_match_oracle(name):
    make, k = CASES[name]
    g = make()
    rg = graphgen.transpose(g) if g.directed else None
    samples = np.asarray(oracle.draw_samples(g.n, k, 3), dtype=np.int32)
    given = None
    if name.startswith("table"):
        given = samples = np.unique(np.concatenate([[0, g.n - 1], samples])).astype(np.int32)
    ref = oracle.estimate_all(g, samples, threads=8, reverse_graph=rg)
    out = LONG if "wide" in name or "limit" in name else OUT
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        for call in range(2):  # the second call enqueues the rounds of the first at once
            print(f"  {g.name}: n={g.n} arcs={g.arcs} k={k} call {call}", flush=True)
            sys.stdout.flush()
            res = cc.cc_estimate(ctx.handle, gh, len(samples), seed=3, samples=given, outputs=out)
            for f in out:
                if f in ref:
                    assert np.array_equal(res[f], np.asarray(ref[f]).astype(res[f].dtype).reshape(res[f].shape)), f
        ctx.release(gh)


def test_patches_errors():
    """A distance past 2^31 - 2 and a node that nothing reaches are still refused."""
    with cc.Context(0) as ctx:
        for w in (4_000_000, (1 << 24) - 2, 1 << 28):  # the last two would wrap inside and between patches
            gh = ctx.upload(_long_path(600, w))
            with pytest.raises(cc.CCError) as e:
                cc.cc_estimate(ctx.handle, gh, 5, seed=1)
            assert e.value.status == cc.CC_EOVERFLOW
            ctx.release(gh)
        i = np.arange(798, dtype=np.int32)
        gh = ctx.upload(graphgen.csr_from_arcs(800, i, i + 1, np.full(798, 7, np.int32)))
        with pytest.raises(cc.CCError) as e:
            cc.cc_estimate(ctx.handle, gh, 5, samples=[3, 9, 200, 400, 700])
        assert e.value.status == cc.CC_EDISCONNECTED
        ctx.release(gh)
        gh = ctx.upload(_grid(20, 30, 1 << 24, 1 << 25))  # the distances fit, the numerators do not
        with pytest.raises(cc.CCError) as e:
            cc.cc_estimate(ctx.handle, gh, 17, seed=3, outputs=OUT)
        assert e.value.status == cc.CC_EOVERFLOW
        ctx.release(gh)


def test_other_calls_on_a_graph_with_patches():
    """The upload numbers such a graph's nodes by patches: reachability
    sampling, node weights and the plain path return the caller's numbering."""
    g = _grid(26, 33)
    beta = graphgen.node_weights(g.n, 5)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        order = np.random.default_rng(2).permutation(g.n).astype(np.int32)
        got = cc.cc_reach_estimate(ctx.handle, gh, 12, order=order)
        ref = oracle.reach_all(g, order, 12, threads=8)
        for f in ref:
            if f in got:
                assert np.array_equal(got[f], np.asarray(ref[f]).astype(got[f].dtype)), f
        w = cc.cc_estimate_weighted(ctx.handle, gh, beta, 30, seed=4)
        wr = oracle.estimate_weighted(g, beta, 30, 4, threads=8)
        assert np.array_equal(w["S_beta"], np.asarray(wr["S_beta"]))
        a = cc.cc_estimate(ctx.handle, gh, 21, seed=6, outputs=("S_hyb", "pivot", "D"))
        b = cc.cc_estimate(ctx.handle, gh, 21, seed=6, mode=cc.CC_PLAIN, outputs=("S_hyb", "pivot", "D"))
        for f in a:
            assert np.array_equal(a[f], b[f]), f
        ctx.release(gh)
