"""Reachability sampling where its searches change their way of working: with
arc lengths, nodes just below and above the number of arcs that a lane group
walks alone, more such nodes in a phase than the list of them holds, and
buckets from one distance wide up; between batches, lists of sources of which
some, most or all have nowhere left to go.  Members, distance sums and positions are
integers and B, R one division of them on both sides: all must be identical."""
import numpy as np
import pytest

import graphgen
import oracle
import paper_1409_0035_amd as cc

pytestmark = pytest.mark.gpu


def _wheels(arms, wheels):
    """Hubs in a row, each with `arms` leaves that lead on to the next hub."""
    src, dst = [], []
    step = arms + 1
    for i in range(wheels):
        h = i * step
        leaves = np.arange(h + 1, h + step)
        src += [np.full(arms, h), leaves]
        dst += [leaves, np.full(arms, (h + step) % (wheels * step))]
    return graphgen.csr_from_arcs(wheels * step, np.concatenate(src), np.concatenate(dst), symmetrize=False,
                                  directed=True)


GRAPHS = {
    "hubs64": lambda: graphgen.with_lengths(_wheels(64, 9), 1, 1000, 1),
    "hubs65": lambda: graphgen.with_lengths(_wheels(65, 9), 1, 1000, 2),
    "hubs257-unit": lambda: graphgen.with_lengths(_wheels(257, 5), 1, 1, 3),
    "hub5000": lambda: graphgen.with_lengths(_wheels(5000, 1), 1, 7, 4),
    "all-hubs": lambda: graphgen.with_lengths(graphgen.gnp(2500, 0.04, 5, directed=True), 1, 3, 5),
    "all-hubs-long": lambda: graphgen.with_lengths(graphgen.gnp(2500, 0.04, 6, directed=True), 1, 100000, 6),
    "grid": lambda: graphgen.grid(37, 41, 8, 0.1, 1, 1000, seed=7),
}


def _check(g, k, inbound):
    order = np.random.default_rng(k).permutation(g.n).astype(np.int32)
    rg = graphgen.transpose(g) if g.directed else None
    ref = oracle.reach_all(g, order, k, inbound=inbound, threads=8, reverse_graph=rg)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        got = cc.cc_reach_estimate(ctx.handle, gh, k, inbound=inbound, order=order)
        for f in ("count", "distsum", "T", "B", "R"):
            assert np.array_equal(got[f], np.asarray(ref[f]).astype(got[f].dtype)), f
        ctx.release(gh)


@pytest.mark.parametrize("inbound", [False, True])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_lengths(name, inbound):
    _check(GRAPHS[name](), 20, inbound)


def _core_and_sinks(core, sinks, chain):
    """A strongly connected core, sinks that hang on it by 1, 8, 9, 512, 513 or all arcs, and chains of
    nodes beside it that stay short of members and end in sinks of their own."""
    rng = np.random.default_rng(core + sinks)
    c = np.arange(core)
    src, dst = [c, c], [np.roll(c, -1), rng.permutation(core)]
    for j, deg in enumerate((1, 8, 9, 512, 513, core)):
        for v in range(core + j, core + sinks, 6 if j < 3 else 600):
            src.append(rng.choice(core, min(deg, core), replace=False))
            dst.append(np.full(src[-1].shape[0], v))
    base = core + sinks
    i = np.arange(chain)
    src += [base + i, np.full(3, 0)]
    dst += [base + np.where(i % 7 == 6, i, np.minimum(i + 1, chain - 1)), base + np.array([0, chain // 2, chain - 1])]
    src, dst = np.concatenate(src), np.concatenate(dst)
    keep = src != dst
    return graphgen.csr_from_arcs(base + chain, src[keep], dst[keep], symmetrize=False, directed=True)


@pytest.mark.parametrize("lengths", [False, True])
@pytest.mark.parametrize("inbound", [False, True])
@pytest.mark.parametrize("core,sinks,chain", [(600, 12000, 3000), (600, 900, 300), (1200, 40, 9000)])
def test_sources_with_nowhere_to_go(core, sinks, chain, inbound, lengths):
    g = _core_and_sinks(core, sinks, chain)
    for k in (1, 5, 100):
        _check(graphgen.with_lengths(g, 1, 9, 2) if lengths else g, k, inbound)
