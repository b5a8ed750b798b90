"""The sums that work groups exchange while a launch runs are read and cleared by
read-modify-writes in the built code too (paper_2512_05460_amd/csrc/pw_chunk.hpp,
compiled here for gfx950): an addition of zero, say, the compiler turns into a
load, which this XCD's cache may answer with an older value."""

import os
import re
import subprocess

import pytest

from paper_2512_05460_amd import build

KERNEL = """
#include "pw_chunk.hpp"
extern "C" __global__ void take_sum(unsigned long long* p, unsigned long long* out)
{
    const pw::i128 v = pw::take_i128(p);
    out[0] = (unsigned long long)v;
    out[1] = (unsigned long long)(v >> 64);
}
"""


def test_sums_are_read_and_cleared_by_read_modify_writes(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    src, out = tmp_path / "words.hip", tmp_path / "words.s"
    src.write_text(KERNEL)
    subprocess.run([hipcc, "-x", "hip", *build._flags(), f"-I{build.CSRC}", "--cuda-device-only", "-S", str(src), "-o",
                    str(out)], check=True, capture_output=True)
    body = re.search(r"^take_sum:(.*?)s_endpgm", out.read_text(), re.M | re.S).group(1)
    assert len(re.findall(r"\bglobal_atomic_swap_x2\b", body)) == 2, body
    assert not re.search(r"\b(global|flat|buffer)_load", body), body
