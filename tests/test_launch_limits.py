"""The largest calls keep to what HIP launches, fewer than 2^32 threads, and their launches cover them once (no GPU needed: the
library's launches meet tests/launch_recorder.c)."""
import os
import subprocess
import sys
import textwrap

import pytest

from paper_2602_08923_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("recorder") / "launch_recorder.so")
    subprocess.check_call(["gcc", "-O1", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.c"), "-o", so])
    return so


def run(recorder, body):
    """`body` in an interpreter of its own, whose library finds the recorder's launches ahead of the runtime's."""
    head = f"""
        import ctypes as C
        class Launch(C.Structure):
            _fields_ = [("grid", C.c_uint32 * 3), ("block", C.c_uint32 * 3), ("args", C.c_uint64 * 4)]
        R = C.CDLL({recorder!r}, mode=C.RTLD_GLOBAL)
        L = C.CDLL({B.LIB_PATH!r})
        P, U = C.c_void_p, C.c_uint64
        def launches():
            a = (Launch * 4096)()
            return a[:R.recorded(a, 4096)]
    """
    got = subprocess.run([sys.executable, "-c", textwrap.dedent(head) + textwrap.dedent(body)], capture_output=True, text=True, timeout=300)
    assert got.returncode == 0, got.stderr


# 16 super-groups to a block of 256 threads: 2^28 are 2^32 threads.  The last: more bf16 super-groups than any memory holds.
@pytest.mark.parametrize("dtype,size", [(0, 4), (1, 2)])
@pytest.mark.parametrize("n", [1, 16, 17, 2 ** 28 - 17, 2 ** 28 - 16, 2 ** 28 - 15, 2 ** 28, 2 ** 28 + 5, 3 * 2 ** 28 + 1, 2 ** 36 + 3])
def test_statistics_of_any_size(recorder, n, dtype, size):
    run(recorder, f"""
        x, mu, F = 1 << 40, 1 << 50, 1 << 54
        L.dq_sg_stats.argtypes = [P, C.c_int, U, P, P, P]
        assert L.dq_sg_stats(x, {dtype}, {n}, mu, F, None) == 0
        at = 0
        for l in launches():
            count = l.args[1]
            assert list(l.args) == [x + at * 256 * {size}, count, mu + 4 * at, F + 4 * at]
            assert list(l.block) == [256, 1, 1] and list(l.grid) == [(count + 15) // 16, 1, 1]
            at += count
        assert at == {n}
    """)
