"""The workgroup sum of the device kernels, compiled for the host one lane at a
time with array bounds checked: a slot per wave for every workgroup size that the
kernels run (three to seven waves)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_16312_amd", "csrc")

# lane 0 of every wave stands for its wave (shuffles bring nothing)
PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)0)
struct Dim { unsigned x; };
static Dim threadIdx{0}, blockIdx{0}, blockDim{THREADS};
static double __shfl_xor(double, int, int) { return 0.0; }
static void __syncthreads() {}
#include "kernels_common.hpp"
int main() {
    double partial[1] = {-1.0}, want = 0.0;
    for (int w = THREADS / 64 - 1; w >= 0; --w) {   // thread 0, which sums, last
        threadIdx.x = 64u * w;
        want += 1 << w;
        dgmg::wg_sum_store<THREADS>((double)(1 << w), partial);
    }
    std::printf("%g %g\n", partial[0], want);
    return 0;
}
"""


@pytest.mark.parametrize("waves", [3, 4, 5, 7])
def test_a_slot_per_wave(tmp_path, waves):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("")
    src = tmp_path / "sum.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "sum"
    subprocess.run(["g++", "-std=c++17", f"-DTHREADS={64 * waves}", "-fsanitize=bounds", "-fno-sanitize-recover=all",
                    "-I", str(tmp_path), "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    got, want = r.stdout.split()
    assert got == want
