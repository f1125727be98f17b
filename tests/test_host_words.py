"""The word forms of the FP64 normal's uniform, cosine and sine, compiled for
the host: bit for bit the values of the forms they replace (the conversion
(m + 1/2) 2^-52 of the top 52 bits, cos_2pi_unit and sin_2pi_unit of that
uniform), over random words and the edges of both folds (all bits clear and
set, and one bit either side of each quarter of the circle)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <hip/hip_runtime.h>
#include <cstdint>
#include <cstdio>
#include <random>
#include "rng.hpp"
static long bad = 0, n = 0;
static void check(uint32_t hi, uint32_t lo)
{
    const uint64_t m = ((uint64_t)hi << 20) | (uint64_t)(lo >> 12);
    const double u = ((double)m + 0.5) * 0x1p-52;
    bad += gmrf::open_uniform_f64(hi, lo) != u;
    bad += gmrf::cos_2pi_words(hi, lo) != gmrf::cos_2pi_unit(u);
    bad += gmrf::sin_2pi_words(hi, lo) != gmrf::sin_2pi_unit(u);
    ++n;
}
int main()
{
    std::mt19937 g(7);
    for (long i = 0; i < 1000000; ++i) {
        const uint32_t hi = g();
        check(hi, g());
    }
    for (uint64_t q = 0; q < 8; ++q)
        for (int64_t d = -2; d <= 2; ++d) {
            const uint64_t w = (q << 61) + ((uint64_t)d << 12);
            check((uint32_t)(w >> 32), (uint32_t)w);
            check((uint32_t)(w >> 32), (uint32_t)w | 0xfffu);
        }
    std::printf("%ld %ld\n", n, bad);
    return 0;
}
"""


def test_word_forms_are_bitwise(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src = tmp_path / "words.hip"
    exe = tmp_path / "words"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-host-only",
                    "-I", os.path.join(ROOT, "paper_1702_05518_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), "-x", "hip", str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    n, bad = subprocess.run([str(exe)], check=True, capture_output=True,
                            text=True).stdout.split()
    assert int(n) > 1_000_000 and int(bad) == 0
