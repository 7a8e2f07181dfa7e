"""Which launches an allocation is, by sizes and by the device's compute units (no GPU needed: the library's launches meet tests/launch_recorder.c, its
questions about the device tests/compute_units.c)."""
import os
import subprocess

import pytest

from test_launch_limits import HERE, run as run_recorded


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("runtime") / "runtime.so")
    sources = [os.path.join(HERE, name) for name in ("launch_recorder.c", "compute_units.c")]
    subprocess.check_call(["gcc", "-O1", "-Wall", "-shared", "-fPIC", *sources, "-o", so])
    return so


def run(runtime, n_cu, body):
    """`body` with so many compute units."""
    run_recorded(runtime, f"""
        C.c_int.in_dll(R, "compute_units").value = {n_cu}
""" + body, 4)


# (J, buckets, max_width, CUs) -> the launches' grids: a block searches for every bucket, or every row's block does; lists in front; positions behind
ONE, ROWS, LISTS = "one", "rows", "lists"


@pytest.mark.parametrize("J,nb,max_width,n_cu,route", [
    (1024, 1, 8, 256, ONE), (1024, 300, 8, 256, ONE), (1025, 1, 8, 256, ROWS), (1025, 128, 8, 256, ROWS), (1025, 129, 8, 256, ONE), (1025, 1, 16, 2, ROWS),
    (1025, 1, 16, 1, ONE), (16384, 16, 16, 256, ROWS), (16384, 17, 16, 256, ONE), (8192, 1, 8, 8, ROWS), (8192, 1, 8, 7, ONE), (40959, 1, 8, 256, ROWS),
    (40960, 1, 8, 256, LISTS), (51200, 1, 16, 256, ROWS), (65536, 4, 8, 256, LISTS), (65536, 5, 8, 256, ONE), (65536, 1, 8, 64, LISTS),
    (51200, 1, 8, 50, LISTS), (51200, 1, 8, 49, ONE), (51200, 2, 8, 64, ONE),   # a partition's CUs: lists would queue
])
def test_routes_of_an_allocation(runtime, J, nb, max_width, n_cu, route):
    rows = -(-J // 1024)
    want = {ONE: [[nb, 1, 1], [rows, nb, 1]], ROWS: [[rows, nb, 1]], LISTS: [[J // 1024, nb, 1], [nb, 1, 1], [rows, nb, 1]]}[route]
    run(runtime, n_cu, f"""
        L.dq_allocate.argtypes = [P, W, W, U, W, P, P, P, P]
        assert L.dq_allocate(1 << 40, {J}, {nb}, {4 * J}, {max_width}, 1 << 50, 1 << 52, 1 << 54, None) == 0
        got = launches()
        assert [list(l.grid) for l in got] == {want}, [list(l.grid) for l in got]
        assert all(list(l.block) == [1024, 1, 1] for l in got)
""")


@pytest.mark.parametrize("J,nb,max_width,n_cu,listed", [
    (40959, 1, 8, 256, 0), (40960, 1, 8, 256, 1), (51200, 5, 8, 256, 1), (51201, 5, 8, 256, 1), (51201, 5, 8, 254, 0), (65536, 4, 8, 256, 1), (65536, 1, 16, 256, 0),
    (51200, 1, 8, 49, 0), (51201, 1, 8, 50, 0), (65537, 1, 8, 256, 0),
])
def test_lists_in_memory_of_their_own_save_a_launch(runtime, J, nb, max_width, n_cu, listed):
    """With as much as dqx_allocate_lists asks for, a launch of every list's block and one of every row's: as many as a search by one block has."""
    run(runtime, n_cu, f"""
        L.dqx_allocate_lists.argtypes, L.dqx_allocate_lists.restype = [W, W, W], U
        assert L.dqx_allocate_lists({J}, {nb}, {max_width}) == {J * nb * listed}
        if {listed}:
            F, widths, pos, counts, lists = 1 << 40, 1 << 50, 1 << 52, 1 << 54, 1 << 55
            L.dqx_allocate_begin.argtypes = [P, W, W, U, W, P, P, P, P, C.c_int, P, P]
            assert L.dqx_allocate_begin(F, {J}, {nb}, {4 * J}, {max_width}, widths, pos, counts, lists, 0, None, None) == 0
            first, second = launches()
            assert list(first.grid) == [{J // 1024}, {nb}, 1] and first.args[0] == F and first.args[3] == lists
            assert list(second.grid) == [{-(-J // 1024)}, {nb}, 1] and second.args[:2] == [F, lists]
            assert L.dqx_allocate_begin(F, {J}, {nb}, {4 * J}, {max_width}, widths, pos, counts, lists + 2, 0, None, None) != 0 and not launches()
""")


@pytest.mark.parametrize("J,nb,max_width,listed", [(1, 1, 8, 0), (1025, 1, 8, 0), (16384, 16, 16, 0), (30000, 2, 8, 0), (40959, 1, 8, 0), (40960, 1, 8, 1), (51200, 1, 16, 0),
                                                   (65536, 4, 8, 1), (65536, 5, 8, 0)])
def test_an_allocation_beside_other_work_searches_on_a_cu_for_each_bucket(runtime, J, nb, max_width, listed):
    """Whether it is given memory for lists or not."""
    grids = [[J // 1024, nb, 1]] * listed + [[nb, 1, 1], [-(-J // 1024), nb, 1]]
    run(runtime, 256, f"""
        L.dqx_allocate_begin.argtypes = [P, W, W, U, W, P, P, P, P, C.c_int, P, P]
        for lists in (None, 1 << 55):
            assert L.dqx_allocate_begin(1 << 40, {J}, {nb}, {4 * J}, {max_width}, 1 << 50, 1 << 52, 1 << 54, lists, 1, None, None) == 0
            assert [list(l.grid) for l in launches()] == {grids}
""")


@pytest.mark.parametrize("J,nb,waves,n_cu,one", [(65536, 1, 5120, 256, 1), (65536, 1, 5120, 70, 1), (65536, 1, 5120, 69, 0), (8192, 1, 2072, 11, 1), (8192, 1, 2072, 10, 0),
                                                 (65537, 1, 5120, 256, 0), (1024, 2, 512, 256, 0)])
def test_an_all_reduce_searches_once_per_row_only_where_each_has_a_cu(runtime, J, nb, waves, n_cu, one):
    run(runtime, n_cu, f"""
        assert L.dqx_searches_and_arranges({J}, {nb}, {waves}) == {one}
""")
