"""The pool of tasks: every interleaving of blocks with unequal counts leaves
the places given without gap or overlap, by the library's own reservation; one
that adds first and takes back is found out by the same check."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2402_00665_amd", "csrc")


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("pool") / "task_pool")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o", out,
                    os.path.join(HERE, "race", "task_pool.cpp")], check=True)
    return out


def explore(binary, args):
    r = subprocess.run([binary, *map(str, args)], capture_output=True, text=True, timeout=120)
    assert r.returncode in (0, 1), r.stderr
    orders, broken = map(int, r.stdout.split())
    return orders, broken


# room, places given at the start, counts
CASES = [(100, 95, 10, 3, 2), (100, 95, 10, 3, 2, 1), (100, 60, 300, 20, 15), (10, 0, 10, 1, 0), (8, 0, 3, 3, 3),
         (100, 100, 1, 0, 7), (100, 90, 9, 1, 1, 10), (5, 4, 2, 1, 1, 3)]


@pytest.mark.parametrize("case", CASES)
def test_every_order_gives_the_places_once(binary, case):
    orders, broken = explore(binary, case)
    assert orders >= 6 and broken == 0


@pytest.mark.parametrize("case", CASES[:3])
def test_an_add_taken_back_is_found_out(binary, case):
    orders, broken = explore(binary, ("--take-back",) + case)
    assert broken > 0


def test_the_cut_reserves_by_it():
    """The kernel that cuts packets takes its places by the tested function
    and moves the pool's counter in no other place."""
    text = open(os.path.join(CSRC, "query_walk.hpp")).read()
    assert "reserve_places(" in text
    assert text.count("&ctrl->tasks") == 1 and "atomicSub" not in text
