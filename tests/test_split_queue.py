"""Slots of the queue that split streams share (csrc/split.hpp), on the CPU:
reservations that fit, end at and pass its last slot, and requests that add
up to more than 2^32 over a call."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("split") / "split_queue")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-I", os.path.join(ROOT, "paper_2210_07580_amd", "csrc"),
                    os.path.join(ROOT, "tests", "split_queue_main.cpp"), "-o", exe], check=True)

    def call(cap, batches, want, before=0):
        r = subprocess.run([exe, str(cap), str(batches), str(want), str(before)], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout
        words = r.stdout.split()
        return int(words[1]), int(words[3]), int(words[5])
    return call


@pytest.mark.parametrize("cap,batches,want", [(0, 3, 1), (1, 3, 1), (7, 3, 2), (8, 4, 2), (8, 5, 2), (100, 1, 101),
                                              (12_000, 90, 5)])
def test_fits_ends_and_passes(run, cap, batches, want):
    fit = min(batches, cap // want)
    assert run(cap, batches, want) == (fit * want, batches - fit, min(cap, batches * want))


def test_requests_of_a_call_beyond_32_bits(run):
    # 400M two-dimensional points, 9e4 per grid, MinPts 1e5: 6.25M batches of
    # 64 queries, 20 neighbours of 44 slices each
    given, alone, used = run(400_000, 6_250_000, 880)
    assert given == 399_520 and alone == 6_250_000 - 454 and used == 400_000


@pytest.mark.parametrize("before", [2**32 - 1, 2**32, 2**33 + 5, 2**51])
def test_a_full_queue_stays_full(run, before):
    assert run(1000, 10, 3, before) == (0, 10, 1000)
