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


def _run(fake_lib, body):
    head = """
        import ctypes, os, sys
        fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before torch's runtime: its functions are found first
        fake.fake_live.restype = fake.fake_peak.restype = ctypes.c_size_t
        fake.fake_allocs.restype = ctypes.c_int64
        fake.fake_fail.argtypes = [ctypes.c_int64, ctypes.c_int64]
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
    code = textwrap.dedent(head) + textwrap.dedent(body)
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
