"""Host-side behaviour on a HIP runtime without a device (fake_hip.c, loaded
ahead of the real one in a child process): what the library allocates, keeps
and sets.  Kernels do not run there, so no results are looked at."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def fake_lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-pthread", "-o", so, os.path.join(HERE, "fake_hip.c")])
    return so


def _run(fake_lib, *body):
    head = """
        import ctypes, os, sys
        fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before torch's runtime: its functions are found first
        fake.fake_live.restype = fake.fake_peak.restype = ctypes.c_size_t
        fake.fake_limit.argtypes = [ctypes.c_size_t]
        import numpy as np
        import graphgen
        import paper_1409_0035_amd as cc

        def lds_log():
            f, s, u, i = ctypes.c_void_p(), ctypes.c_int64(), ctypes.c_int64(), 0
            while fake.fake_lds(i, ctypes.byref(f), ctypes.byref(s), ctypes.byref(u)):
                yield f.value, s.value, u.value
                i += 1

        ctx = cc.Context(0)
    """
    code = textwrap.dedent(head) + "".join(textwrap.dedent(b) for b in body)
    p = subprocess.run([sys.executable, "-c", code, fake_lib], cwd=ROOT, timeout=110, capture_output=True, text=True)
    assert p.returncode == 0, p.stdout + p.stderr


def test_lds_limit_of_a_kernel_is_one_value(fake_lib):
    """The limit belongs to the kernel, and serving slots launch from several
    threads: every call sets the same one, so that no thread's smaller graph
    can lower it between another's set and launch."""
    _run(fake_lib, """
        for n in (30_000, 49_000, 20_000):
            gh = ctx.upload(graphgen.ba(n, 4, seed=1))
            try:
                cc.cc_estimate(ctx.handle, gh, 16, seed=1)
            except cc.CCError:  # nothing ran
                pass
            ctx.release(gh)
        limit, launches = {}, 0
        for f, was_set, used in lds_log():
            if was_set >= 0:
                assert limit.setdefault(f, was_set) == was_set, "limits differ"
            else:
                assert used <= limit[f]
                launches += 1
        assert launches >= 3
    """)


# bytes a weighted graph keeps on the device: row bounds, ends, lengths, the two id maps, one word where a list of hub
# chunks is empty, (end, length) pairs; with the arcs reversed once more for a digraph
WEIGHTED_BYTES = """
        def weighted_bytes(g):
            one = 4 * (g.n + 1) + 4 * g.arcs + 4 * g.arcs + 8 * g.arcs
            return one * (2 if g.directed else 1) + 2 * 4 * g.n + (8 if g.directed else 4)
"""


def test_upload_without_memory_for_patches(fake_lib):
    """The patch tables are an optimisation: where memory holds the graph but
    not them, the graph is accepted without, and nothing of the attempt stays."""
    _run(fake_lib, WEIGHTED_BYTES, """
        und = graphgen.grid(60, 70, 8, 0.1, 1, 1000, seed=1)
        for g in (und, graphgen.with_lengths(graphgen.symmetric_digraph(graphgen.grid(60, 70, 4)), 1, 50, 8)):
            need, before = weighted_bytes(g), fake.fake_live()
            for spare in (0, 1, 10_000, 50_000, 150_000):  # the tables take more
                fake.fake_limit(before + need + spare)
                gh = ctx.upload(g)
                assert fake.fake_live() - before == need, (g.directed, spare)
                ctx.release(gh)
                assert fake.fake_live() == before
            fake.fake_limit(before + need - 1)
            try:
                ctx.upload(g)
                raise SystemExit("a graph without room was accepted")
            except cc.CCError as e:
                assert e.status == cc.CC_ENOMEM
            assert fake.fake_live() == before
    """)


def test_upload_keeps_the_patch_tables_it_uses(fake_lib):
    """Of an undirected graph: patch bounds and ids, slots, the outside arcs
    (none here: nothing counted them) with their bounds, cursors and three
    counters, and the neighbours -- not the reversed arcs, nor the slots'
    owners, which only the build reads."""
    _run(fake_lib, WEIGHTED_BYTES, """
        g, before = graphgen.grid(16, 32, 8, 0.1, 1, 1000, seed=1), fake.fake_live()
        gh = ctx.upload(g)
        patches = [np_ for np_ in range(2, 12) if fake.fake_live() - before - weighted_bytes(g) ==
                   4 * (np_ + 1) + 4 * g.n + 32 * 256 * np_ + 4 * (3 * (np_ + 1) + 2) + 16 + 8 * 32 * np_]
        assert len(patches) == 1, fake.fake_live() - before - weighted_bytes(g)
        ctx.release(gh)
        assert fake.fake_live() == before
    """)


def test_served_jobs_stay_inside_the_budget(fake_lib):
    """Admission charges a job what it will hold: with room for one search by
    patches (17 MB at 256 samples, whatever the graph's size), or for one small
    graph's estimate with its error outputs, four slots run one at a time."""
    _run(fake_lib, """
        ctx.close()
        # (graph, samples, outputs, bytes of one estimate's buffers within a few rounded up to whole MiB)
        cases = [(graphgen.grid(16, 32, 8, 0.1, 1, 1000, seed=1), 256, ("S_hyb",), 20 << 20),
                 (graphgen.ba(1000, 4, seed=1), 256, ("S_hyb", "S_err"), 6 << 20)]
        for g, k, outputs, one in cases:
            fake.fake_sync_us(0)
            with cc.Context(0, mem_budget_bytes=one, max_inflight=4) as c:
                gh = c.upload(g)
                before = fake.fake_live()
                fake.fake_reset_peak()
                fake.fake_sync_us(3000)
                jobs = [cc.cc_submit(c.handle, gh, k, seed=j, outputs=outputs) for j in range(6)]
                for j in jobs:
                    try:
                        cc.cc_wait(j)
                    except cc.CCError:  # nothing ran
                        pass
                    cc.cc_job_release(j)
                held = fake.fake_peak() - before
                assert held <= one, (g.name, held, one)
                c.release(gh)
    """)
