"""The 8-byte block entries of the sign-table kernels and the places of their nodes,
on the host (paper_2512_05460_amd/csrc/pw_signtab.hpp, compiled with g++): degrees
are taken from their binary32 reciprocals, exactly below 2^20, and every node lies
where its run of equal degree says."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from synth import graphs

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2512_05460_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("entries") / "sign_entry_check")
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", os.path.join(HERE, "native", "sign_entry_check.cpp"),
                    "-o", exe], check=True)

    def run(lines):
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
        return [ln.split() for ln in out.splitlines()]
    return run


def test_degrees_below_2_20(check):
    assert check(["degrees 1 1048576"]) == [["ok"]]


def test_nodes_lie_where_their_runs_say(check):
    rng = np.random.default_rng(11)
    cases = [np.sort(np.diff(graphs.workload_graph(k).row_ptr))[::-1].tolist() for k in ("ba1k", "cl100k")]
    cases += [[1, 1], [2] * 1000, [5, 4, 3, 2, 1], [70000] + [3] * 70000, [2] * 512 + [1] * 2, list(range(300, 0, -1))]
    for _ in range(20):
        cases.append(np.sort(rng.zipf(1.8, size=int(rng.integers(1, 5000))).clip(1, 3000))[::-1].tolist())
    res = check(["order " + " ".join(str(v) for v in (len(d), *d)) for d in cases])
    assert len(res) == len(cases) and all(r[0] == "ok" for r in res), [r for r in res if r[0] != "ok"]
