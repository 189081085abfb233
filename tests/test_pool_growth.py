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
