// Layout of the contraction operands (plain C++, so that host code can check
// the address arithmetic of the kernels).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define TWA_HD __host__ __device__ __forceinline__
#else
#define TWA_HD inline
#endif

namespace twa {

// The constant operand A of a contraction (P rows, K columns) is stored
// stage-blocked: the kt columns of K stage q of all P rows are contiguous,
// row after row, and the stages follow one another.  One LDS stage of MT rows
// is then a single contiguous run of MT * kt elements (whole cache lines),
// where a row-major matrix would give MT runs of kt elements one row pitch
// apart.  kt = K elements per LDS stage of the tile configuration.
// In the split form (Prec::NP parts per value) a stage holds the kt columns
// of all P rows of part 0, then those of part 1: element (i, j) of part p.
TWA_HD int64_t a_index(int64_t i, int64_t j, int64_t P, int64_t kt, int np = 1, int p = 0) {
    return ((j / kt) * np + p) * P * kt + i * kt + (j % kt);
}

// Operand column of component a (0 = x, 1 = y) of trajectory k: x and y of
// 16 consecutive trajectories sit in two adjacent 16-column blocks, so one
// lane of an MFMA output pair holds both components of one (spin, trajectory).
TWA_HD int64_t opcol(int64_t k, int a) { return 32 * (k >> 4) + 16 * a + (k & 15); }

// The column operand X of a contraction (C2 columns) is stage-blocked the same
// way: element i of column c, part p, with the kt elements of one K stage of
// all columns contiguous.  A stage's columns of a tile are then one contiguous
// run (a row-major operand gave runs of one stage's 64 or 128 bytes, half a
// cache line at 64), and 16 neighbouring columns written by one epilogue block
// share cache lines.
TWA_HD int64_t x_index(int64_t c, int64_t i, int64_t C2, int64_t kt, int np = 1, int p = 0) {
    return ((i / kt) * np + p) * C2 * kt + c * kt + i % kt;
}

// An epilogue block stores rows row .. row + 15 (row a multiple of 16) of the
// 32 columns of 16 trajectories, four rows of one column per lane.  A stage and
// a part lie C2 kt elements apart, which 32-bit byte offsets do not reach for
// large ensembles, so they go into the 64-bit base of the block's descriptor:
// the element where the block's columns (from col = opcol(k, 0)) of the stage
// of `row` start; from there the lane's first element is less than
// op_block_span away.  With kt = 8 (FP64) lanes 32 .. 63 are one stage on: they
// take the base of row + 8.
TWA_HD int64_t op_block(int64_t row, int64_t col, int64_t C2, int64_t kt, int np, int part) {
    return ((row / kt) * np + part) * C2 * kt + col * kt;
}
TWA_HD uint32_t op_lane(int lane, int c, int64_t row, int kt) {
    return (uint32_t)((16 * c + (lane & 15)) * kt + (int)((row + 4 * (lane >> 4)) % kt));
}
TWA_HD constexpr int op_block_span(int kt) { return 32 * kt; }

}  // namespace twa
