"""Where the step kernels' epilogues store operand values, for ensembles of any
size: the 64-bit base of a block's descriptor plus the lane's 32-bit offset is
the element that the layout names, the offset never leaves the descriptor, and
both hold where a K stage of all columns is more than 4 GiB away from the next
(from 6.7 million trajectories on).  twa_index.h is plain C++ and is compiled
for the host here."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "twa_index.h"
#include <cstdio>
using namespace twa;
int main() {
    struct { int size, kt, np; } formats[] = {{8, 8, 1}, {8, 16, 1}, {4, 16, 1}, {4, 32, 1}, {2, 32, 1}, {2, 64, 1},
                                              {2, 32, 2}, {2, 64, 2}};
    const int64_t B[] = {16, 128, 6710912, 11184816, 33554432, 134217728, (int64_t)1 << 33};
    long checked = 0, far = 0;
    for (auto f : formats)
        for (int64_t Bp : B)
            for (int64_t row = 0; row < 400; row += 16)
                for (int64_t k = 0; k < Bp; k += Bp / 16 * 5 / 16 * 16 + 16)
                    for (int c = 0; c < 2; ++c)
                        for (int lane = 0; lane < 64; ++lane)
                            for (int part = 0; part < f.np; ++part) {
                                const int64_t C2 = 2 * Bp;
                                const int64_t at = f.kt >= 16 || lane < 32 ? row : row + 8;
                                const int64_t base = op_block(at, opcol(k, 0), C2, f.kt, f.np, part);
                                const uint32_t off = op_lane(lane, c, row, f.kt);
                                for (int r = 0; r < 4; ++r) {
                                    const int64_t want = x_index(opcol(k + (lane & 15), c), row + 4 * (lane >> 4) + r,
                                                                 C2, f.kt, f.np, part);
                                    if (base + off + r != want || (int)off + r >= op_block_span(f.kt)) {
                                        std::printf("kt %d parts %d B %lld row %lld k %lld lane %d\n", f.kt, f.np,
                                                    (long long)Bp, (long long)row, (long long)k, lane);
                                        return 1;
                                    }
                                    ++checked;
                                }
                                // what one 32-bit offset from the wave's first row could not reach
                                if (row % 64 && (x_index(opcol(k, c), row, C2, f.kt, f.np, part) -
                                                 x_index(opcol(k, c), row / 64 * 64, C2, f.kt, f.np, 0)) *
                                                        f.size > 0xFFFFFFFFll)
                                    ++far;
                            }
    std::printf("%ld elements, %ld blocks past 32 bits\n", checked, far);
    return far > 0 ? 0 : 2;
}
"""


def test_operand_stores_reach_any_ensemble(tmp_path):
    src, exe = tmp_path / "index.cpp", tmp_path / "index"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2608_10075_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_step_kernels_store_operands_through_these_bases():
    """No block offset that grows with the ensemble is left in 32 bits."""
    text = open(os.path.join(ROOT, "paper_2608_10075_amd", "csrc", "twa_step_impl.h")).read()
    assert "op_block(rw, col, C2, KT, NP, q)" in text and "op_lane(lane, c, row, KT)" in text
    for line in text.splitlines():
        if "(uint32_t)" in line:
            assert "C2" not in line and "Bp" not in line, line
