"""Small graphs are searched by one workgroup per sample: every output at the
edges of that path (64-node chunks, words of 64 samples, arcs copied to LDS or
not, frontiers longer than their list, hubs, distances up to 254 and beyond,
sums of a round trip) against the oracle.  Integers and the estimates' doubles
are exact integers divided once on both sides, so they must be identical."""
import sys

import numpy as np
import pytest

import graphgen
import oracle
import paper_1409_0035_amd as cc

pytestmark = pytest.mark.gpu
OUT = ("S_hyb", "S_samp", "S_piv", "S_pub", "pivot", "delta", "sampsum", "src_sum", "samples", "dmat", "D", "S_err",
       "S_ad", "S_ad_err")

CASES = {
    "path1": (lambda: graphgen.path(1), 1),
    "path2": (lambda: graphgen.path(2), 2),
    "path63": (lambda: graphgen.path(63), 63),
    "path65": (lambda: graphgen.path(65), 65),
    "path255-254-levels": (lambda: graphgen.path(255), 3),
    "path256-deeper": (lambda: graphgen.path(256), 256),
    "star5000": (lambda: graphgen.star(5000), 129),
    "K300": (lambda: graphgen.complete(300), 192),
    "ba1000-k256": (lambda: graphgen.ba(1000, 4, seed=1), 256),
    "ba7001-arcs-in-lds": (lambda: graphgen.ba(7001, 4, seed=2), 65),
    "ba8200-arcs-in-memory": (lambda: graphgen.ba(8200, 4, seed=3), 64),
    "dense-long-rows": (lambda: graphgen.gnp(1500, 0.2, 4), 17),
    "grid-thin-frontier": (lambda: graphgen.grid(9, 200, 4), 50),
    "ba49152-largest": (lambda: graphgen.ba(49152, 4, seed=5), 9),
    "ba49153-general-path": (lambda: graphgen.ba(49153, 4, seed=5), 9),
    "dcycle254": (lambda: graphgen.directed_cycle(254), 4),
    "dcycle255-deeper": (lambda: graphgen.directed_cycle(255), 4),
    "rmat11dir-arcs-in-lds": (lambda: graphgen.rmat(11, 8, seed=6, directed=True), 100),
    "rmat14dir": (lambda: graphgen.rmat(14, 16, seed=7, directed=True), 130),
}


@pytest.mark.parametrize("name", list(CASES))
def test_small_graph_matches_oracle(name):
    make, k = CASES[name]
    g = make()
    rg = graphgen.transpose(g) if g.directed else None
    samples = np.asarray(oracle.draw_samples(g.n, k, 3), dtype=np.int32)
    ref = oracle.estimate_all(g, samples, threads=8, reverse_graph=rg) if g.n <= 10_000 else \
        oracle.estimate_tails(g, samples, threads=8, reverse_graph=rg)
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        for call in range(2):  # the second call finds the first one's buffers
            print(f"  {g.name}: n={g.n} arcs={g.arcs} k={k} call {call}", flush=True)
            sys.stdout.flush()
            res = cc.cc_estimate(ctx.handle, gh, k, seed=3, outputs=OUT)
            for f in OUT:
                if f in ref:
                    assert np.array_equal(res[f], np.asarray(ref[f]).astype(res[f].dtype).reshape(res[f].shape)), f
        ctx.release(gh)


def test_small_graph_not_connected_leaves_outputs():
    """A node that no sample reaches: CC_EDISCONNECTED, device outputs untouched."""
    import torch
    g = graphgen.csr_from_arcs(700, np.arange(0, 698, dtype=np.int32), np.arange(1, 699, dtype=np.int32))
    with cc.Context(0) as ctx:
        gh = ctx.upload(g)
        out = {"S_hyb": torch.full((g.n,), -7.0, dtype=torch.float64, device="cuda"),
               "pivot": torch.full((g.n,), -7, dtype=torch.int32, device="cuda"),
               "src_sum": torch.full((40,), -7, dtype=torch.int64, device="cuda")}
        for mode in (cc.CC_BATCHED, cc.CC_BATCHED | cc.CC_GRAPH):
            with pytest.raises(cc.CCError) as e:
                cc.cc_estimate_device(ctx.handle, gh, 40, out, mode=mode, seed=2)
            assert e.value.status == cc.CC_EDISCONNECTED
        torch.cuda.synchronize()
        for t in out.values():
            assert bool((t == -7).all())
        ctx.release(gh)


def test_batch_of_graphs_past_the_small_path():
    """Undirected graphs of more than 49,152 nodes still share one traversal
    in cc_estimate_batch: every output equals the job run alone."""
    fields = ("S_hyb", "S_piv", "pivot", "delta", "sampsum", "dmat")
    with cc.Context(0) as ctx:
        hs = [ctx.upload(graphgen.ba(n, 4, seed=n)) for n in (49_153, 60_001, 1000)]
        jobs = [(h, k, 5 + k) for h, k in zip(hs, (64, 100, 16))]
        got, sts = cc.cc_estimate_batch(ctx.handle, jobs, outputs=fields)
        assert sts == [cc.CC_OK] * 3
        for (h, k, seed), r in zip(jobs, got):
            alone = cc.cc_estimate(ctx.handle, h, k, seed=seed, outputs=fields)
            for f in fields:
                assert np.array_equal(r[f], alone[f]), (k, f)
        for h in hs:
            ctx.release(h)
