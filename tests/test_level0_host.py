"""The scan of small tables on the CPU, in its own source compiled for the host under
AddressSanitizer: the interval search (csrc/fdy_level0.hpp) against the definition over every small
table, and the chunk states (csrc/fdy_flat_state.hpp) over sequences of launches."""
import os
import subprocess

import pytest

from paper_2604_06664_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("level0") / "level0_host")
    subprocess.check_call([build.hipcc(), "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g",
                           "-Xarch_host", "-fsanitize=address", "-fno-gpu-sanitize",
                           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(HERE, "level0", "level0_host.hip"), "-o", exe])
    return exe


def run(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    return r.stdout


def test_small_tables(program):
    assert ", 0 wrong" in run(program, "valid")


def test_invalid_tables_stay_in_bounds(program):
    assert ", 0 wrong" in run(program, "invalid")


def test_both_ways_to_stage_leave_the_same(program):
    assert ", 0 wrong" in run(program, "staging")


def test_chunk_states_of_launches_in_turn(program):
    assert ", 0 wrong" in run(program, "states")
