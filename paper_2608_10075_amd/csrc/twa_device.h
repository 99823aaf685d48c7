// Device-side building blocks: counter-based noise, number formats of the
// contraction, and the MFMA fragments used by the step kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/twa.h"
#include "twa_index.h"

namespace twa {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two 32x32
// -> 64-bit multiplies with the published multipliers, the key advanced by
// the published Weyl increments between rounds.
struct U4 {
    uint32_t x, y, z, w;
};

__device__ __forceinline__ U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // each product as one 64-bit value: one v_mad_u64_u32 instead of a
        // v_mul_hi_u32 and a v_mul_lo_u32 (both quarter rate)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = U4{(uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0};
    }
    return c;
}

// Counter words: (slot, trajectory, step, tag | point << 8).
enum : uint32_t { TAG_PUMP = 0u, TAG_COLLECTIVE = 1u, TAG_INIT = 2u };

// Box-Muller (Box & Muller 1958) on two words.  u1 = ((a >> 8) + 1) 2^-24 in
// (0, 1] and u2 = (b >> 8) 2^-24 are exact in binary32.  Binary32 uses the
// hardware transcendentals: v_log_f32 (log2; ln u1 = ln 2 log2 u1),
// v_sqrt_f32, and v_sin_f32 / v_cos_f32, which take their argument in
// revolutions (sin 2 pi u2 directly, u2 in [0, 1)).
__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, float& z0, float& z1) {
    const float u1 = (float)((a >> 8) + 1u) * 5.9604644775390625e-08f;
    const float u2 = (float)(b >> 8) * 5.9604644775390625e-08f;
    const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));
    z0 = r * __builtin_amdgcn_cosf(u2);
    z1 = r * __builtin_amdgcn_sinf(u2);
}
__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, double& z0, double& z1) {
    const double u1 = (double)((a >> 8) + 1u) * 5.9604644775390625e-08;
    const double u2 = (double)(b >> 8) * 5.9604644775390625e-08;
    const double r = sqrt(-2.0 * log(u1));
    double s, c;
    sincospi(2.0 * u2, &s, &c);
    z0 = r * c;
    z1 = r * s;
}

// ---------------------------------------------------------------------------
// number formats
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

struct bf16s {
    uint16_t v;
};

// round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int PREC>
struct Prec;

template <>
struct Prec<TWA_PREC_FP64> {
    static constexpr int NP = 1;      // bf16 parts per operand value
    static constexpr int NSW = 1;     // sweeps over a K block
    typedef double G;   // contraction operand
    typedef double S;   // state / accumulator
    typedef f64x4 AV;
    // The f64 16x16x4 MFMA returns row (lane/16) + 4 r in register r; feeding
    // A-operand row m with spin 4 (m % 4) + m / 4 makes register r of lane l
    // hold spin 4 (l/16) + r, the layout of the other formats.
    __device__ static __forceinline__ int arow(int m) { return 4 * (m & 3) + (m >> 2); }
    __device__ static __forceinline__ G to_g(S v) { return v; }
    __device__ static __forceinline__ void mma(AV& c, const uint4& a, const uint4& b) {
        const f64x2 fa = __builtin_bit_cast(f64x2, a), fb = __builtin_bit_cast(f64x2, b);
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[0], fb[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[1], fb[1], c, 0, 0, 0);
    }
};

template <>
struct Prec<TWA_PREC_FP32> {
    static constexpr int NP = 1;
    static constexpr int NSW = 1;
    // 16x16 MFMA output: register r of lane l holds row 4 (l/16) + r
    __device__ static __forceinline__ int arow(int m) { return m; }
    typedef float G;
    typedef float S;
    typedef f32x4 AV;
    __device__ static __forceinline__ G to_g(S v) { return v; }
    __device__ static __forceinline__ void mma(AV& c, const uint4& a, const uint4& b) {
        const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
        for (int q = 0; q < 4; ++q) c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[q], fb[q], c, 0, 0, 0);
    }
};

template <>
struct Prec<TWA_PREC_BF16> {
    static constexpr int NP = 1;
    static constexpr int NSW = 1;
    // 16x16 MFMA output: register r of lane l holds row 4 (l/16) + r
    __device__ static __forceinline__ int arow(int m) { return m; }
    typedef bf16s G;
    typedef float S;
    typedef f32x4 AV;
    __device__ static __forceinline__ G to_g(S v) { return G{f32_to_bf16_rne(v)}; }
    __device__ static __forceinline__ void mma(AV& c, const uint4& a, const uint4& b) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                    0, 0, 0);
    }
};

template <>
struct Prec<TWA_PREC_FP16> {
    static constexpr int NP = 1;
    static constexpr int NSW = 1;
    // 16x16 MFMA output: register r of lane l holds row 4 (l/16) + r
    __device__ static __forceinline__ int arow(int m) { return m; }
    typedef _Float16 G;
    typedef float S;
    typedef f32x4 AV;
    __device__ static __forceinline__ G to_g(S v) { return (_Float16)v; }
    __device__ static __forceinline__ void mma(AV& c, const uint4& a, const uint4& b) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                   0, 0);
    }
};

// Split BF16: every operand value x is stored in two bf16 parts, hi = bf16(x)
// and lo = bf16(x - hi), and one accumulator takes NSW = 3 sweeps over each K
// block of P values, A.hi X.hi, then A.hi X.lo, then A.lo X.hi; the dropped
// lo lo and the rounding of lo are O(2^-17) relative.  (All three products of
// a K stage formed together load each part once, 4 reads in place of 6, and
// took 266 us a step at 4096 x 512 against 318, but add up in another
// order; where <S+S-> nearly cancels, g2 and its standard error then differ in
// the fourth digit, beyond any rounding of the outputs themselves.)
template <>
struct Prec<TWA_PREC_BF16X3> : Prec<TWA_PREC_BF16> {
    static constexpr int NP = 2;
    static constexpr int NSW = 3;
};

// the bf16 parts of a value
template <int NP>
__device__ __forceinline__ void bf16_parts(float v, uint16_t (&h)[NP]) {
    h[0] = f32_to_bf16_rne(v);
#pragma unroll
    for (int p = 1; p < NP; ++p) {
        v -= bf16_to_f32(h[p - 1]);
        h[p] = f32_to_bf16_rne(v);
    }
}

// one operand value: p[0], or in the split form its parts blk elements apart
template <int PREC>
__device__ __forceinline__ void put_op(typename Prec<PREC>::G* p, int64_t blk, typename Prec<PREC>::S v) {
    constexpr int NP = Prec<PREC>::NP;
    if constexpr (NP > 1) {
        uint16_t h[NP];
        bf16_parts<NP>(v, h);
#pragma unroll
        for (int q = 0; q < NP; ++q) p[q * blk].v = h[q];
    } else {
        p[0] = Prec<PREC>::to_g(v);
    }
}

// element (i, j) of a stage-blocked constant operand, all its parts
template <int PREC>
__device__ __forceinline__ void put_a(typename Prec<PREC>::G* A, int64_t i, int64_t j, int64_t P, int64_t kt,
                                      typename Prec<PREC>::S v) {
    constexpr int NP = Prec<PREC>::NP;
    put_op<PREC>(A + a_index(i, j, P, kt, NP, 0), P * kt, v);
}

// element i of column c of a column operand, all its parts
template <int PREC>
__device__ __forceinline__ void put_x(typename Prec<PREC>::G* X, int64_t c, int64_t i, int64_t C2, int64_t kt,
                                      typename Prec<PREC>::S v) {
    put_op<PREC>(X + x_index(c, i, C2, kt, Prec<PREC>::NP, 0), C2 * kt, v);
}

// four elements i .. i + 3 (i % 4 == 0, so they share a K stage) of column c
// of a column operand, all their parts, one store each (FP64 two)
template <int PREC>
__device__ __forceinline__ void put_x4(typename Prec<PREC>::G* X, int64_t c, int64_t i, int64_t C2, int64_t kt,
                                       const typename Prec<PREC>::S (&v)[4]) {
    constexpr int NP = Prec<PREC>::NP;
    typename Prec<PREC>::G* p = X + x_index(c, i, C2, kt, NP, 0);
    if constexpr (PREC == TWA_PREC_FP64) {
        reinterpret_cast<double2*>(p)[0] = make_double2(v[0], v[1]);
        reinterpret_cast<double2*>(p)[1] = make_double2(v[2], v[3]);
    } else if constexpr (NP > 1) {
        uint16_t h[4][NP];
#pragma unroll
        for (int r = 0; r < 4; ++r) bf16_parts<NP>(v[r], h[r]);
#pragma unroll
        for (int q = 0; q < NP; ++q)
            *reinterpret_cast<ushort4*>(p + q * C2 * kt) = make_ushort4(h[0][q], h[1][q], h[2][q], h[3][q]);
    } else if constexpr (PREC == TWA_PREC_FP32) {
        *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        uint16_t h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = __builtin_bit_cast(uint16_t, Prec<PREC>::to_g(v[r]));
        *reinterpret_cast<ushort4*>(p) = make_ushort4(h[0], h[1], h[2], h[3]);
    }
}

// The normals of one step: zeta^{x,y} of every (trajectory, spin) into the
// noise rows of the column operand, g^{x,y} of every trajectory.  A block of
// NT threads takes one K stage of NT / (kt / 4) neighbouring trajectories, four
// spins of one trajectory to a thread: its stores fill whole runs of kt
// elements of neighbouring columns, 8 bytes a lane (one spin a thread stored 2
// bytes at a time: 4.8 us a launch at N x B = 201 x 500, 16.9 at 1000 x 4096).
// Rows past N of the last stage stay zero.
template <int NT>
__host__ __device__ inline int64_t noise_blocks(int64_t N, int64_t B, int64_t kt) {
    const int64_t tpb = NT / (kt / 4);
    return ((N + kt - 1) / kt) * ((B + tpb - 1) / tpb);
}
template <int PREC, int NT>
__device__ __forceinline__ void noise_block(uint32_t blk, int64_t N, int64_t B, int64_t P, int64_t Bp, int kt,
                                            uint32_t k0, uint32_t k1, uint32_t point, uint32_t n,
                                            typename Prec<PREC>::G* Xop, typename Prec<PREC>::S* g) {
    typedef typename Prec<PREC>::S S;
    const uint32_t nst = (uint32_t)((N + kt - 1) / kt), qs = (uint32_t)kt / 4;
    const uint32_t stg = blk % nst, tid = threadIdx.x;
    const int64_t k = (int64_t)(blk / nst) * (NT / qs) + tid / qs, i = (int64_t)stg * kt + 4 * (tid % qs);
    if (k >= B || i >= N) return;
    S x[4], y[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const U4 w = philox4x32_10(U4{(uint32_t)(i / 2) + h, (uint32_t)k, n, TAG_PUMP | (point << 8)}, k0, k1);
        box_muller(w.x, w.y, x[2 * h], y[2 * h]);
        box_muller(w.z, w.w, x[2 * h + 1], y[2 * h + 1]);
    }
#pragma unroll
    for (int r = 1; r < 4; ++r)
        if (i + r >= N) x[r] = y[r] = S(0);
    put_x4<PREC>(Xop, opcol(k, 0), P + i, 2 * Bp, kt, x);
    put_x4<PREC>(Xop, opcol(k, 1), P + i, 2 * Bp, kt, y);
    if (i == 0) {
        const U4 v = philox4x32_10(U4{0u, (uint32_t)k, n, TAG_COLLECTIVE | (point << 8)}, k0, k1);
        S g0, g1;
        box_muller(v.x, v.y, g0, g1);
        g[k] = g0;
        g[Bp + k] = g1;
    }
}

}  // namespace twa
