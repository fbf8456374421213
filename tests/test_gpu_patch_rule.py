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
