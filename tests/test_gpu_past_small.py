"""The bit-parallel levels, their captures and replays, knobs, error outputs,
borrowed graphs, batches and the allocation-free lane, on the graphs of the
modules below: those tests run here once more with 2^21 loops at node 0 of
every unit-length graph they upload.  Loops change no distance and no estimate,
and the oracle sees the graph without them, but they put it past the small
graphs' line, behind which the same call would run one workgroup per sample
instead of the code that these tests are about.  Every estimate's search is
looked at, and one that reports a single launch has to be a replay."""
import numpy as np
import pytest

import paper_1409_0035_amd as cc
from test_gpu_batch import (test_batch_matches_single_runs, test_batch_with_jobs_that_run_alone_or_fail,  # noqa: F401
                            test_serving_batches_small_jobs)
from test_gpu_borrow import (test_borrowed_device_outputs_and_replays, test_borrowed_equals_uploaded_and_oracle,  # noqa: F401
                             test_borrowed_reach_and_serving)
from test_gpu_errest import (test_error_estimates_in_a_batch, test_error_estimates_match_oracle,  # noqa: F401
                             test_sweep_only_outputs)
from test_gpu_graph import (test_host_outputs_accept_graph_flag, test_replays_match_eager,  # noqa: F401
                            test_replays_with_error_outputs, test_replays_write_samples,
                            test_round_trip_replays_match_oracle)
from test_gpu_parity import (test_ba10k_k64_full, test_closed_form_families, test_device_outputs_on_torch_stream,  # noqa: F401
                             test_directed_rmat_round_trip, test_ragged_sample_counts, test_random_configurations,
                             test_random_small_graphs, test_round_trip_row_widths,
                             test_worked_example_path9)
from test_gpu_tuning import (test_autotune_keeps_results, test_bfs_knobs_do_not_change_results,  # noqa: F401
                             test_merge_grid_not_a_multiple_of_64)
from test_zz_no_alloc import test_noalloc_matches_estimate_device  # noqa: F401

pytestmark = pytest.mark.gpu
LOOPS = 1 << 21


@pytest.fixture(scope="module")
def ctx():
    c = cc.Context(0)
    yield c
    c.close()


@pytest.fixture(autouse=True)
def past_the_small_path(monkeypatch):
    upload, borrow = cc.cc_graph_upload, cc.cc_graph_borrow_device
    kept, searches, padded = [], [], []

    def padded_upload(ctx, n, arcs, row_ptr, col_idx, w=None, flags=0):
        if w is None:
            row_ptr = np.concatenate([[0], np.asarray(row_ptr, dtype=np.int64)[1:] + LOOPS])
            col_idx = np.concatenate([np.zeros(LOOPS, np.int32), np.asarray(col_idx, dtype=np.int32)])
            arcs += LOOPS
            padded.append(n)
        return upload(ctx, n, arcs, row_ptr, col_idx, w, flags)

    def padded_borrow(ctx, n, arcs, row_ptr, col_idx, w=None, flags=0):
        if w is None:
            import torch
            row_ptr, col_idx = row_ptr + LOOPS, torch.cat([col_idx.new_zeros(LOOPS), col_idx])
            row_ptr[0] = 0
            torch.cuda.synchronize()
            kept.append((row_ptr, col_idx))  # read in place for the graph's life
            arcs += LOOPS
        return borrow(ctx, n, arcs, row_ptr, col_idx, w, flags)

    def watched(name):
        call = getattr(cc, name)

        def run(ctx, *args, **kw):
            out = call(ctx, *args, **kw)
            t = cc.cc_last_timing(ctx)
            assert t["search"] in (cc.CC_SEARCH_LEVELS, cc.CC_SEARCH_PLAIN, cc.CC_SEARCH_WEIGHTED,
                                   cc.CC_SEARCH_PATCHES) or t["search"] & cc.CC_SEARCH_REPLAY, t["search"]
            assert (t["launches"] == 1) <= bool(t["search"] & cc.CC_SEARCH_REPLAY or
                                                t["search"] == cc.CC_SEARCH_WEIGHTED)
            searches.append(t["search"])
            return out

        monkeypatch.setattr(cc, name, run)

    monkeypatch.setattr(cc, "cc_graph_upload", padded_upload)
    monkeypatch.setattr(cc, "cc_graph_borrow_device", padded_borrow)
    watched("cc_estimate")
    watched("cc_estimate_device")
    yield
    assert searches or padded  # a batch alone reports no timing
