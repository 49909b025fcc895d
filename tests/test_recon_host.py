"""The forward pass forms the optical depths that the backward pass forms again: its
short form of the bounds gives the adjoint's value to the last bit, on centred
measures, off-centre ones, and ones whose atoms nearly coincide (there a zero counted
or chosen before its last Newton step would move a whole weight). csrc/recon.h is
compiled for the CPU, with exact reciprocals and square roots."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# what recon.h and common.h take from the HIP headers
HIP_HEADER = """#pragma once
#include <cmath>
#include <cstring>
using std::isfinite;
#define __host__
#define __device__
#define __forceinline__ inline
#define __cosf cosf
static struct { unsigned x; } threadIdx;
"""


def test_forward_bound_is_the_adjoints(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs a host C++ compiler")
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_HEADER)
    exe = str(tmp_path / "recon_host")
    subprocess.run([gxx, "-O2", "-std=c++17", f"-I{tmp_path}", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_2512_11800_amd/csrc", os.path.join(ROOT, "tests", "recon_host.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=110).stdout
    print(out)
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 9 and all(int(r[2]) == 640_000 for r in rows)
    assert [r for r in rows if int(r[3]) != 0] == []
