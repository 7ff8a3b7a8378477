"""The sizes that the non-allocating PCG accepts: 48 + max(ceil(N / 256), ceil(cells /
(256 / b))) doubles of 131,072, for every block size, in whatever form the level is held."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_16312_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "internal.hpp"
int main() {
    long long n;
    int b;
    while (std::scanf("%lld %d", &n, &b) == 2)
        std::printf("%d\n", dgmg::noalloc_doubles(n * b, n, b) <= dgmg::kScratchLimit);
    return 0;
}
"""


def test_accepted_sizes(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    cases = []
    for b in (4, 8, 9, 16, 25, 27, 64):
        top = (131072 - 48) * (256 // b)       # every workgroup full
        cases += [(n, b) for n in (1, top // 2, top - 1, top, top + 1, top + 256 // b, 2 * top)]
    r = subprocess.run([str(exe)], input="".join(f"{n} {b}\n" for n, b in cases), capture_output=True, text=True, check=True)
    want = [48 + max(-(-n * b // 256), -(-n // (256 // b))) <= 131072 for n, b in cases]
    assert [bool(int(v)) for v in r.stdout.split()] == want
    assert want.count(False) == 21 and want.count(True) == 28
