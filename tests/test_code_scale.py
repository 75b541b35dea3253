"""td_code_scale (codes.h), compiled for the CPU: the codes that one fma gives with the scale of a row are those of the definition,
rint(w / s) with s = max / 127 in 64 bits, for every pair of bf16 mantissas and every quotient down to 2^-20."""
import shutil
import subprocess

import pytest

from paper_2501_10054_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "codes.h"

static int code(float w, float m) {
    const double s = (double)m / 127.0;
    return (int)std::fmin(std::fmax(std::rint((double)w / s), -127.0), 127.0);
}

int main() {
    long count = 0;
    for (int e : {-99, -30, 0, 31, 98})
        for (int b = 128; b < 256; ++b) {
            const float m = std::ldexp((float)b, e - 7), scale = td_code_scale(m, code(0.5f * m, m));
            for (int down = 0; down <= 20; ++down)
                for (int a = 0; a < 256; ++a)
                    for (int sign : {-1, 1}) {
                        const float w = sign * std::ldexp((float)a, e - 7 - down);
                        if (std::fabs(w) > m) continue;
                        if ((int8_t)(td_code_bits(w, scale) & 255u) != code(w, m)) {
                            std::printf("%g of %g: %d\n", w, m, code(w, m));
                            return 1;
                        }
                        ++count;
                    }
        }
    std::printf("%ld\n", count);
    return 0;
}
"""


def test_codes_of_every_pair_of_mantissas(tmp_path):
    clang = next((c for c in (shutil.which("amdclang++"), "/opt/rocm/bin/amdclang++", shutil.which("clang++")) if c and shutil.which(c)), None)
    if clang is None:
        pytest.skip("no clang")
    src, exe = tmp_path / "codes.cpp", tmp_path / "codes"
    src.write_text(PROGRAM)
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 6_000_000
