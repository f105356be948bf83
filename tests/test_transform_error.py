"""Rounding of the transforms of csrc/fft.hpp, on the CPU: compiled for the host, their error on
random FP32 lines is no larger than that of the direct form (a product per input, then sums and
differences), for every line length and number of elements per thread of the kernels."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2012_04838_amd", "csrc")
# what fft.hpp takes from the device compiler; one thread, so its barriers are empty
DEVICE = """#pragma once
#define __device__
#define __host__
#define __forceinline__ inline
struct Index { int x; };
static Index threadIdx{0}, blockDim{1};
inline void __syncthreads() {}
inline void __builtin_amdgcn_fence(int, const char*) {}
inline void __builtin_amdgcn_wave_barrier() {}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_fp32_transform_error_is_no_larger_than_the_direct_form(tmp_path):
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(DEVICE)
    exe = str(tmp_path / "transform_error")
    # products and sums contract to fused multiply-adds, as on the device
    subprocess.run(["g++", "-std=c++17", "-O2", "-march=native", "-ffp-contract=fast", "-w", "-I", str(tmp_path),
                    "-I", CSRC, os.path.join(HERE, "transform_error.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    rows = [line.split() for line in out.splitlines()]
    assert len(rows) == 3 + 7 * 4 + 2
    for n, e, inv, err, direct in rows:
        # one rounding of 2^-24 per level and component at the least would be 6e-8
        assert 1e-8 < float(direct) < 2e-7
        assert float(err) <= float(direct), f"N={n} E={e} inverse={inv}: {err} against {direct}"
