"""Where the products with four wavefronts load from: td_find_slice (slices.h), compiled for the CPU and run over whole
sequences.  Every slice of either pair of operands is fetched once, and no load reaches past an operand's rows - also if
the hardware's range check, offset >= num_records - soff, is taken to wrap."""
import os
import shutil
import subprocess

import pytest

from paper_2501_10054_amd import build as B

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "slices.h"

constexpr int SL = 128;
static long cases = 0;

// one operand's loads: rows x (k, k2) bytes, tiles of TM rows
template <bool REPAIR> static void check(int rows, int TM, uint32_t k, uint32_t k2, int splits, int ks, int rot, int rot2, int ahead) {
    const int nk1 = (int)(k / SL), nk2 = (int)(k2 / SL), per = (nk1 + nk2 + splits - 1) / splits, s0 = ks * per;
    int nk = nk1 + nk2 - s0;
    nk = nk < 0 ? 0 : nk > per ? per : nk;
    if (rot > 0 && rot >= (REPAIR ? nk1 : nk)) return;
    if (rot2 > 0 && rot2 >= nk2) return;
    const td_slices q{nk1, nk2, s0, nk, rot, rot2, k, k2};
    const td_i32x4 r1 = {1, 0, (int)((uint32_t)rows * k), 7}, r2 = {2, 0, (int)((uint32_t)rows * k2), 7};
    std::vector<int> seen(nk1 + nk2, 0);
    td_slice_source o{};
    o.rs.w = 7;
    for (int t = 0; t < nk + ahead; ++t) {
        o.t = t;
        for (int step = 0; step < 6; ++step) td_find_slice<REPAIR, SL>(o, q, r1, r2, step);
        const bool second = o.rs.x == 2;
        bool fetched = false;
        for (int row = 0; row < TM; ++row)
            for (uint32_t piece = 0; piece < SL; piece += 16) {
                const uint32_t offset = (uint32_t)row * o.pitch + piece;
                if (offset >= (uint32_t)o.rs.z - o.soff) continue;              // out of range: nothing is read
                fetched = true;
                const uint64_t end = (uint64_t)o.soff + offset + 16, size = (uint64_t)rows * (second ? k2 : k);
                if (end > size || row >= rows) {
                    std::printf("slice %d of %d: row %d of %d, bytes to %llu of %llu\n", t, nk, row, rows, (unsigned long long)end, (unsigned long long)size);
                    std::exit(1);
                }
            }
        if (fetched != (t < nk)) {
            std::printf("slice %d of %d is %s\n", t, nk, fetched ? "fetched" : "not fetched");
            std::exit(1);
        }
        if (t < nk) ++seen[(second ? nk1 : 0) + (int)(o.soff / SL)];
    }
    for (int s = 0; s < nk1 + nk2; ++s)
        if (seen[s] != (s >= s0 && s < s0 + nk)) {
            std::printf("slice %d fetched %d times\n", s, seen[s]);
            std::exit(1);
        }
    ++cases;
}

int main() {
    for (int rows : {1, 100, 256})
        for (uint32_t slices : {1u, 2u, 5u, 16u})
            for (uint32_t more : {0u, 16u}) {                                    // (a ragged row: its rest is not in the sequence)
                for (int splits : {1, 2, 8})
                    for (int ks = 0; ks < splits; ++ks)
                        for (int rot : {0, 1, 7}) {
                            check<false>(rows, 256, slices * SL + more, 0, splits, ks, rot, 0, 7);
                            check<false>(rows, 256, 4 * SL, slices * SL + more, splits, ks, rot, 0, 7);
                        }
                for (int rot : {0, 1, 7})
                    for (int rot2 : {0, 1, 7}) check<true>(rows, 256, slices * SL, 2 * slices * SL, 1, 0, rot, rot2, 7);
            }
    std::printf("%ld\n", cases);
}
"""


def test_loads_stay_inside_the_operands(tmp_path):
    clang = next((c for c in (shutil.which("amdclang++"), "/opt/rocm/bin/amdclang++", shutil.which("clang++")) if c and os.path.exists(c)), None)
    if clang is None:
        pytest.skip("no clang (slices.h uses its vector types)")
    src, exe = tmp_path / "slices.cpp", tmp_path / "slices"
    src.write_text(PROGRAM)
    subprocess.run([clang, "-x", "c++", "-std=c++17", "-O1", "-I", B.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 300
