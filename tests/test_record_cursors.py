"""Cursor words of the deposit records (ctd_records.h): the protocol played on
the CPU with random interleavings, from counts about to leave 32 bits on."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIGH = 1 << 31


@pytest.fixture(scope="module")
def play(tmp_path_factory):
    exe = tmp_path_factory.mktemp("records") / "record_check"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_1109_3266_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "record_check.cpp"), "-o", str(exe)],
                   check=True)

    def run(*line):
        r = subprocess.run([str(exe)], input=" ".join(map(str, line)) + "\n", text=True,
                           capture_output=True, check=True, timeout=60)
        return r.stdout.strip()
    return run


def test_segments_fill_and_run_out(play):
    for seed in range(6):
        for lanes, deposits, segments in [(1, 700, 2), (8, 300, 3), (200, 30, 4), (64, 50, 0)]:
            assert play(seed, lanes, deposits, segments, 1, HIGH) == "ok"


# the count passes the mark in the middle of the play or has passed it (the end
# of 32 bits is 2^31 adds past the mark, and each burst of adds that ends before
# then is wound back)
@pytest.mark.parametrize("start", [HIGH - 40, HIGH, HIGH + 5, (1 << 32) - 20_000])
def test_count_is_wound_back(play, start):
    for seed in range(6):
        for lanes in (1, 7, 300):
            assert play(seed, lanes, 50, 0, start, HIGH) == "ok"


def test_a_count_never_wound_back_is_caught(play):
    assert play(1, 7, 50, 0, (1 << 32) - 40, 0) != "ok"
