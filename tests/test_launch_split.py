"""Host arithmetic of split launches (csrc/launch_split.h), built and run on the CPU: HIP takes no grid
of 2^32 lanes or more, whatever the launch knobs allow."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2210_10246_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path_factory.mktemp("split") / "launch_split_host")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-O1", "-o", exe,
                    os.path.join(HERE, "launch_split_host.cpp")], check=True, timeout=300)
    return lambda *args: [int(x) for x in subprocess.run(
        [exe, *map(str, args)], capture_output=True, text=True, check=True, timeout=60).stdout.split()]


def test_no_launch_has_2_32_lanes(program):
    knob = 65536                                    # the largest and default cap per compute unit
    for threads in (64, 128, 256, 512, 1024):
        for units in (1, 256, 304, 1024):
            groups, = program(units * knob, threads)
            assert groups * threads < 1 << 32
            assert groups == units * knob or (groups + 1) * threads >= 1 << 32   # and no fewer than need be
    assert program(256, 256, 256 * knob, 128, 256 * knob, 256) == [256, 1 << 24, (1 << 24) - 1]


def test_the_attention_launches_are_bounded_by_it():
    """Each place that turns the attention knobs (keys 4 and 5) into a number of workgroups."""
    with open(os.path.join(CSRC, "attention.hip")) as f:
        text = f.read()
    caps = re.findall(r"const int64_t cap = ([^;]*);", text)
    assert [("most_groups(" in c) for c in caps if "bpc" in c or "blocks_per_cu" in c] == [True] * 3


@pytest.mark.parametrize("total,cap", [(1, 1), (7, 3), (9, 3), (256, 257), (257, 256), ((1 << 32) - 1, (1 << 24) - 1)])
def test_split_covers_every_workgroup_once(program, total, cap):
    *pairs, ok = program("split", total, cap, 1 << 40)
    firsts, counts = pairs[::2], pairs[1::2]
    assert ok == 1
    assert firsts == [sum(counts[:i]) for i in range(len(counts))]
    assert sum(counts) == total and 0 < min(counts) and max(counts) <= cap


def test_split_ends_at_the_first_refused_launch(program):
    assert program("split", 10, 4, 4) == [0, 4, 4, 4, 0]
    assert program("split", 10, 4, 0) == [0, 4, 0]
