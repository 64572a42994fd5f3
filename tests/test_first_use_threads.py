"""The first calls of several host threads that need a kernel's dynamic-LDS limit raised, a raising that fails, and which
launches a call makes: the library against stand-ins for the HIP runtime's entry points (tests/first_use_threads.cpp), on the CPU."""
import os
import subprocess

import pytest

from paper_2511_15927_amd import binding as bd

HERE = os.path.dirname(os.path.abspath(__file__))
ERR_HIP = -6


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("first_use") / "first_use_threads")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-pthread", "-I", os.path.join(os.path.dirname(HERE), "include"),
                    os.path.join(HERE, "first_use_threads.cpp"), "-o", exe, "-ldl"], check=True)

    def run(*args):
        r = subprocess.run([exe, bd.LIB_PATH, *map(str, args)], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [int(v) for v in r.stdout.split()]
    return run


@pytest.mark.parametrize("entry", ["fwd", "bwd", "block", "m2", "m2_block"])
def test_a_second_thread_does_not_launch_under_a_limit_still_being_raised(program, entry):
    first, second, launches, refused, _ = program("race", entry)
    assert (first, second, refused) == (0, 0, 0) and launches >= 2


# (the raising that fails, and what was launched before it: the preparations and the direction that parks, into the workspace)
@pytest.mark.parametrize("entry,failing,before", [("fwd", 1, 0), ("bwd", 1, 1), ("block", 1, 0), ("m2_block", 1, 0),
                                                  ("m2", 1, 0), ("m2", 2, 1), ("m2", 3, 2)])
def test_a_failed_raising_is_reported_and_tried_again(program, entry, failing, before):
    first, second, launches, refused, of_first = program("fail", entry, failing)
    assert (first, second, refused, of_first) == (ERR_HIP, 0, 0, before) and launches > of_first


def test_time_parts_are_kept_where_only_z_and_out_rows_are_far_apart(program):
    """The preparation, the state pass, its carry and a walk per direction; with x rows as far apart the call runs in one part.  (And the
    conv tail's commit.)"""
    assert program("fail", "m2_far", 0) == [0, 0, 12, 0, 6]
    assert program("fail", "m2_far_x", 0) == [0, 0, 8, 0, 4]
