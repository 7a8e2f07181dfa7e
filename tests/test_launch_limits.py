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


def run(recorder, body, args):
    """`body` in an interpreter of its own, whose library finds the recorder's launches ahead of the runtime's."""
    head = f"""
        import ctypes as C
        class Launch(C.Structure):
            _fields_ = [("grid", C.c_uint32 * 3), ("block", C.c_uint32 * 3), ("args", C.c_uint64 * 8)]
        R = C.CDLL({recorder!r}, mode=C.RTLD_GLOBAL)
        L = C.CDLL({B.LIB_PATH!r})
        P, U, W = C.c_void_p, C.c_uint64, C.c_uint32
        C.c_int.in_dll(R, "args_taken").value = {args}
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
            assert l.args[:4] == [x + at * 256 * {size}, count, mu + 4 * at, F + 4 * at]
            assert list(l.block) == [256, 1, 1] and list(l.grid) == [(count + 15) // 16, 1, 1]
            at += count
        assert at == {n}
    """, 4)


# A search has 1,024 threads to a bucket: 2^22 buckets are 2^32 threads.  Buckets above 65,536 super-groups take another kernel.
@pytest.mark.parametrize("J,n", [(1, 1), (1, 65535), (1, 65536), (5, 2 ** 22 - 1), (5, 2 ** 22), (1025, 2 ** 22 + 7), (65537, 65537)])
@pytest.mark.parametrize("width", [8, 16])
def test_allocation_of_any_number_of_buckets(recorder, J, n, width):
    run(recorder, f"""
        J, F, widths, pos, counts = {J}, 1 << 40, 1 << 50, 1 << 52, 1 << 54
        L.dq_allocate.argtypes = [P, W, W, U, W, P, P, P, P]
        assert L.dq_allocate(F, J, {n}, 4 * J, {width}, widths, pos, counts, None) == 0
        at = 0
        for l in launches():
            assert list(l.block) == [1024, 1, 1] and l.args[0] == F + 4 * J * at and l.args[1] & 0xFFFFFFFF == J
            positions = J <= 65536 and l.args[3] == counts + 20 * at
            if positions:                                            # behind the search of the same buckets
                assert list(l.grid) == [(J + 1023) // 1024, searched, 1]
            else:
                assert l.args[2] == 4 * J and list(l.grid)[1:] == [1, 1]
                if J <= 65536:
                    assert l.args[3] == pos + 4 * J * at
                searched = l.grid[0]
            if positions or J > 65536:
                at += searched
        assert at == {n}
    """, 4)


# A thread per super-group.
@pytest.mark.parametrize("n", [1, 256, 257, 2 ** 32 - 257, 2 ** 32 - 256, 2 ** 32 - 255, 2 ** 32, 2 ** 33 + 1])
def test_combination_of_any_size(recorder, n):
    run(recorder, f"""
        mu_all, F_all, mu, F = 1 << 40, 1 << 50, 1 << 52, 1 << 54
        L.dq_stats_combine.argtypes = [P, P, W, U, P, P, P]
        assert L.dq_stats_combine(mu_all, F_all, 3, {n}, mu, F, None) == 0
        at = 0
        for l in launches():
            assert l.args[0] == mu_all + 4 * at and l.args[1] == F_all + 4 * at and l.args[2] & 0xFFFFFFFF == 3
            count = l.args[4]
            assert l.args[3] == {n} and l.args[5] == mu + 4 * at and l.args[6] == F + 4 * at
            assert list(l.block) == [256, 1, 1] and list(l.grid) == [(count + 255) // 256, 1, 1]
            at += count
        assert at == {n}
    """, 7)
