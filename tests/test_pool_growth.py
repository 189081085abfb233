"""Host rules of the particle pool's growth, compiled without a device."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
POOL, RECORD, COUNT, TEMP = 1, 2, 4, 8


@pytest.fixture(scope="module")
def need(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pool") / "pool_growth")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-o", exe, os.path.join(HERE, "helpers", "pool_growth.cpp")],
                   check=True, capture_output=True)

    def run(*row):
        r = subprocess.run([exe], input=" ".join(map(str, row)), capture_output=True, text=True, check=True)
        return int(r.stdout)
    return run


@pytest.mark.parametrize("also", [0, TEMP, RECORD | TEMP])
def test_a_step_without_room_is_taken_again_whatever_else_it_raised(need, also):
    assert need(POOL | also, 1 << 21, 1 << 24, 2000000, 100000) == 2100000
    assert need(POOL | also, 1 << 21, 2100000, 2000000, 100000) == 2100000


@pytest.mark.parametrize("row", [(0, 1 << 21, 1 << 24, 2000000, 100000), (TEMP, 1 << 21, 1 << 24, 2000000, 100000),
                                 (COUNT, 1 << 21, 1 << 24, 10, 10), (POOL, 1 << 21, 2099999, 2000000, 100000),
                                 (POOL, 1 << 24, 1 << 24, 1 << 24, 1), (POOL | TEMP, 1, 1 << 29, 1 << 28, 1 << 62)])
def test_other_errors_and_full_pools_are_not(need, row):
    assert need(*row) == 0


def _total(slots):
    return sum((slots * per + 255) // 256 * 256 for per in (8, 4, 8, 8, 4, 8))


@pytest.fixture(scope="module")
def move(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pool") / "pool_move")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined", "-o", exe,
                    os.path.join(HERE, "helpers", "pool_move.cpp")], check=True, capture_output=True)

    def run(have, n, need, cap, budget, taken=0, bad=0):
        r = subprocess.run([exe, *map(str, (have, n, need, cap, budget, taken, bad))], capture_output=True, text=True,
                           check=True)
        return tuple(map(int, r.stdout.split()))
    return run


DONE, NO_MEMORY, FAILED, LOST = range(4)


@pytest.mark.parametrize("n", [0, 1, 1000])
def test_growth_takes_the_largest_size_that_fits_beside_the_pool(move, n):
    have, need, cap = 1000, 1100, 100000
    for size in (4000, 1375, 1100):
        assert move(have, n, need, cap, _total(have) + _total(size)) == (DONE, size, 1, 0, _total(size))
    assert move(have, n, 3900, 3950, 1 << 30) == (DONE, 3950, 1, 0, _total(3950))


def test_growth_makes_room_through_the_host_where_both_do_not_fit(move):
    have, n, need, cap = 1000, 1000, 1100, 100000
    for size in (1100, 1375):
        assert move(have, n, need, cap, _total(size)) == (DONE, size, 1, 6, _total(size))
    # a pool of nearly all of the device, up to its capacity
    assert move(90000, 90000, 99999, 100000, _total(100000)) == (DONE, 100000, 1, 6, _total(100000))


def test_growth_that_cannot_fit_leaves_the_pool(move):
    have, n, need, cap = 1000, 1000, 1100, 100000
    assert move(have, n, need, cap, _total(1100) - 1) == (NO_MEMORY, have, 1, 0, _total(have))
    # others take the rest while the pool is in host memory: it comes back at its size
    assert move(have, n, need, cap, _total(1100), taken=_total(1100) - _total(have)) == (NO_MEMORY, have, 1, 6, _total(have))
    assert move(have, n, need, cap, _total(1100), taken=_total(1100) - _total(have) + 1)[:3] == (LOST, have, -1)


@pytest.mark.parametrize("bad", [1, 3])
def test_a_failed_copy_leaves_the_pool(move, bad):
    assert move(1000, 1000, 1100, 100000, 1 << 30, 0, bad)[:3] == (FAILED, 1000, 1)
    assert move(1000, 1000, 1100, 100000, _total(1100), 0, bad)[:3] == (FAILED, 1000, 1)
