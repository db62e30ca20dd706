"""The block sweep's LDS arithmetic (csrc/sweep_index.h) on the CPU: for every number of
tile rows, step and slot, with a tile or without one, the operands a wavefront reads lie in
the LDS that the launch asks for, and in the part they are meant to be in."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "sweep_index.h"
using namespace arb;
int main() {
    const int block = 16 * kSwLd, reach = 15 * kSwLd + 3 + 12;  // furthest lane, last product
    for (int nb = 1; nb <= 16; ++nb) {
        const SweepLds L = sweep_lds(nb);
        if (L.end * 8 > 160 * 1024 || L.end < kSwMaxWaves * block) return 1;
        for (int k = 0; k < nb; ++k)
            for (int i = 0; i <= nb; ++i)
                for (int j = 0; j <= i; ++j) {
                    const bool none = i == nb;
                    const int ti = none ? kSwNone : i, tj = none ? kSwNone : j;
                    const int a = sweep_operand_a(L, nb, ti), b = sweep_operand_b(L, nb, ti, tj, k);
                    if (a < 0 || b < 0 || a + reach >= L.end || b + reach >= L.end) {
                        std::printf("nb %d step %d tile %d %d: %d %d of %d\n", nb, k, ti, tj, a, b,
                                    L.end);
                        return 2;
                    }
                    if (none) continue;
                    if (a != L.W + i * block) return 3;
                    const int want = i != k ? (k & 1) * L.buf + j * block
                                   : j != k ? L.W + j * block : L.T + (k & 1) * block;
                    if (b != want) return 4;
                }
    }
    return 0;
}
"""


def test_operands_stay_in_the_lds(tmp_path):
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2107_10800_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", inc, str(src), "-o", str(exe)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
