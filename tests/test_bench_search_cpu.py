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
