"""The vote for the launch shape of a batch on sign tables, on the host
(paper_2512_05460_amd/csrc/pw_signtab.hpp, compiled with g++): the shape that
most work asks for, and never one that no query asks for."""

import itertools
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2512_05460_amd", "csrc")


def test_shape_is_one_that_was_asked_for(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "shape_vote_check")
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", os.path.join(HERE, "native", "shape_vote_check.cpp"),
                    "-o", exe], check=True)
    cases = []
    for m in (1, 2, 3):
        for shapes in itertools.product(range(4), repeat=m):
            for work in itertools.product((0.0, 1.0, 5.0), repeat=m):
                cases.append(list(zip(shapes, work)))
    lines = "\n".join(" ".join(str(v) for v in (len(c), *(x for pair in c for x in pair))) for c in cases)
    out = subprocess.run([exe], input=lines + "\n", capture_output=True, text=True, check=True).stdout.split()
    assert len(out) == len(cases)
    for c, got in zip(cases, map(int, out)):
        sums = {}
        for shape, work in c:
            sums[shape] = sums.get(shape, 0.0) + work
        assert got in sums and sums[got] == max(sums.values()), (c, got)
