"""Host logic of the benchmark: the weighted roofline names the kernel that the
library says it ran (no GPU)."""
import bench
import paper_1409_0035_amd as cc

TUNING = {"delta": 750}


def _timing(search, launches):
    return dict(kernel_launches=launches, kernel_ms=1.0, arcs_scanned=1000, nodes_visited=100, search=search)


def test_weighted_roofline_names_the_search_that_ran():
    two = [_timing(cc.CC_SEARCH_WEIGHTED, 2)] * 3  # a round trip, or two groups of samples: two launches an estimate
    assert bench.wsearch_roofline(two, "none", 100, 700, 4, TUNING)["kernel"] == "k_wsearch"
    rounds = [_timing(cc.CC_SEARCH_PATCHES, 40)] * 3
    assert bench.wsearch_roofline(rounds, "none", 100, 700, 4, TUNING)["kernel"] == "k_patch_round"


def test_small_graph_roofline_counts_the_arcs_read():
    t = dict(kernel_ms=0.04, arcs_scanned=2_000_000, search=cc.CC_SEARCH_SMALL)
    r = bench.small_roofline([t, t], 64)
    assert r["kernel"] == "k_small_search" and r["launches_per_step"] == 1
    assert r["achieved"] == 200.0 and r["arcs_per_sample"] == 31250.0
