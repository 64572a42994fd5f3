"""The first calls of several host threads that need a kernel's dynamic-LDS limit raised, and a raising that fails: the
library against stand-ins for the HIP runtime's entry points (tests/first_use_threads.cpp), on the CPU."""
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

    def run(mode, entry):
        r = subprocess.run([exe, bd.LIB_PATH, mode, entry], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [int(v) for v in r.stdout.split()]
    return run


@pytest.mark.parametrize("entry", ["fwd", "bwd"])
def test_a_second_thread_does_not_launch_under_a_limit_still_being_raised(program, entry):
    first, second, launches, refused = program("race", entry)
    assert (first, second, refused) == (0, 0, 0) and launches >= 2


@pytest.mark.parametrize("entry", ["fwd", "bwd"])
def test_a_failed_raising_is_reported_and_tried_again(program, entry):
    first, second, launches, refused = program("fail", entry)
    assert (first, second, refused) == (ERR_HIP, 0, 0) and launches >= 1
