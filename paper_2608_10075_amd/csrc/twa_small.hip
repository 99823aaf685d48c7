// Fused small-N path of the TWA trajectories (Eq. (S1), SM Sec. S1): for
// short chains the per-step work is a few N x N products per trajectory, far
// too little to fill the device per launch, so the multi-kernel step is bound
// by its launches.  One launch integrates every step: a workgroup owns T = 8 CB
// trajectories for the whole run, with
//   * NB = ceil(N / 16) compute waves, wave w holding the 16 rows of spins
//     16 w .. 16 w + 15 of -dt/2 W and of -sqrt(dt) F in registers and the
//     spins themselves in the MFMA output layout; the spin vectors are
//     exchanged through LDS, and every wave sums them for the collective term
//     of Eq. (S1) from the operands it reads anyway;
//   * four producer waves that draw the next steps' noise into LDS and form
//     the window moments of the steps before, off the compute waves' path.
// Bound by the per-step chain exchange -> MFMA -> update -> exchange ->
// MFMA -> update of the compute waves (MFMA issue from N of about 50 on).
// From N = 17 on every sum is formed in the order of the stage kernels on the
// tiles they take for that N (16 rows to N = 48, then 64), so in FP32 a run
// gives the same bits on either path (to N = 16 the noise field is added first).
// Heun and the semi-implicit midpoint scheme; FP64 or FP32 state, operands and
// MFMA.  Noise from the same Philox counters as the multi-kernel path.
// The shortest chains have a kernel of their own, lanes_run_kernel.
#include <algorithm>
#include <cmath>


#include "twa_device.h"
#include "twa_internal.h"

namespace twa {
namespace {

constexpr int PRODUCERS = 4;   // producer waves per workgroup
constexpr int LANES_THREADS = 256;

template <typename S>
struct Small;
template <>
struct Small<float> {
    static constexpr int MAX_NB = 8;    // rows of A' and F: 8 NB registers per lane
    static constexpr int PAD = 4;       // spins of padding per LDS vector: 16 bytes, so columns start on other banks
    typedef f32x4 V;
    __device__ static __forceinline__ int arow(int m) { return m; }
    __device__ static __forceinline__ V mfma(float a, float b, V c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};
template <>
struct Small<double> {
    static constexpr int MAX_NB = 4;    // 16 NB registers per lane
    static constexpr int PAD = 2;
    typedef f64x4 V;
    // operand row m feeds spin 4 (m % 4) + m / 4, so that output register r of
    // lane l is spin 4 (l / 16) + r as in binary32
    __device__ static __forceinline__ int arow(int m) { return 4 * (m & 3) + (m >> 2); }
    __device__ static __forceinline__ V mfma(double a, double b, V c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
};

template <typename S>
__device__ __forceinline__ void kahan(S& sum, S& comp, S v) {
    const S y = v - comp;
    const S t = sum + y;
    comp = (t - sum) - y;
    sum = t;
}

// the value of the lane 8 columns away within a row of 16 lanes
__device__ __forceinline__ float ror8(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x128, 0xf, 0xf, true));
}
__device__ __forceinline__ double ror8(double v) {
    const int2 h = __builtin_bit_cast(int2, v);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(h.x, 0x128, 0xf, 0xf, true),
                                                __builtin_amdgcn_mov_dpp(h.y, 0x128, 0xf, 0xf, true)));
}

// v plus the value of the lane 16 (32) lanes away: rows of 16 lanes pairwise, then halves
__device__ __forceinline__ float across16(float v) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ float across32(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ __forceinline__ double across16(double v) {
    const uint2 h = __builtin_bit_cast(uint2, v);
    const auto x = __builtin_amdgcn_permlane16_swap(h.x, h.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(h.y, h.y, false, false);
    return __builtin_bit_cast(double, make_uint2(x[0], y[0])) + __builtin_bit_cast(double, make_uint2(x[1], y[1]));
}
__device__ __forceinline__ double across32(double v) {
    const uint2 h = __builtin_bit_cast(uint2, v);
    const auto x = __builtin_amdgcn_permlane32_swap(h.x, h.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(h.y, h.y, false, false);
    return __builtin_bit_cast(double, make_uint2(x[0], y[0])) + __builtin_bit_cast(double, make_uint2(x[1], y[1]));
}

// Sum over the spins of a column in the order of the stage kernels: lane group
// g adds its rows 4 g .. 4 g + 3 of the 16-row blocks of a wave of theirs (one
// block to N = 48, two beyond), the four groups are added, then the waves of a
// tile (one, two) and the tiles.  add() takes the blocks in order; total() is
// the same in all lanes of a column.
template <typename S, int NB>
struct ColumnSum {
    static constexpr int RB = NB > 3 ? 2 : 1, NW = (NB + RB - 1) / RB;
    S ps[NW];
    template <typename V>
    __device__ __forceinline__ void add(const int q, const V& v) {
        S p = q % RB ? ps[q / RB] : S(0);
#pragma unroll
        for (int r = 0; r < 4; ++r) p += v[r];
        ps[q / RB] = p;
    }
    __device__ __forceinline__ S total() const {
        S s = 0;
#pragma unroll
        for (int w = 0; w < NW; w += RB) {
            S t = S(0) + across32(across16(ps[w]));
            if (RB == 2 && w + 1 < NW) t += across32(across16(ps[w + 1]));
            s += t;
        }
        return s;
    }
};

// orders a wave's own LDS accesses (which the hardware executes in order) for
// the compiler
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename S>
struct SmallArgs {
    int n;                    // atoms
    int64_t B, P, Bp;
    const double *W, *F;
    double cw, cf;            // -dt/2, -sqrt(dt)
    S c1, c2;                 // Gamma dt / 2, sqrt(Gamma dt)
    uint32_t k0, k1, point;
    int64_t n_steps, burnin;
    int sib;
    const S* s_in;
    S *s_out, *mom;
};

// CB column blocks of 16: CB = 2 holds the x and y components of 16
// trajectories in one block each; CB = 1 those of 8 in the two halves of one
// block (the lanes of a pair exchange their fields and both carry the spin).
// U steps per batch of noise: with one compute wave nothing but the noise
// crosses waves, so waves meet once per batch of 8 steps; else every step.
template <typename S, int NB, int CB>
__global__ __launch_bounds__(64 * (NB + PRODUCERS)) void small_run_kernel(SmallArgs<S> a) {
    typedef Small<S> K;
    typedef typename K::V V;
    constexpr int T = 8 * CB, COLS = 16 * CB, XP = 16 * NB + K::PAD, U = NB == 1 ? 8 : 1;
    constexpr int ZB = NB == 1 ? PRODUCERS : 2;
    __shared__ __attribute__((aligned(16))) S Xs[COLS][XP];     // state, x and y columns
    __shared__ __attribute__((aligned(16))) S Xd[COLS][XP];     // predictor increment
    __shared__ __attribute__((aligned(16))) S Xp[NB == 1 ? 1 : COLS][XP];   // predictor (NB > 1)
    __shared__ __attribute__((aligned(16))) S Xz[NB == 1 ? 1 : T][XP];      // state, z (NB > 1, for the window moments)
    __shared__ __attribute__((aligned(16))) S Z[ZB][COLS][XP];  // pump normals (NB = 1: one per producer)
    __shared__ S Gn[NB == 1 ? PRODUCERS : 2][T][2];             // collective normals
    __shared__ __attribute__((aligned(16))) S Q[NB == 1 ? 2 * U : 1][NB == 1 ? COLS : 1][XP];   // noise fields (NB = 1)
    __shared__ S R[2][U][NB == 1 ? 4 : 1][3][T];                // partial spin sums of the steps of a batch (NB = 1)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = lane & 15, g = lane >> 4, n = a.n;
    const int64_t kb = (int64_t)blockIdx.x * T;      // first trajectory
    const int64_t SP = a.Bp * a.P;
    const bool compute = wave < NB;
    const int w = compute ? wave : 0;

    for (int t = tid; t < ZB * COLS * XP; t += 64 * (NB + PRODUCERS)) (&Z[0][0][0])[t] = S(0);

    // rows of the operands (lane: row c, columns 16 q + 4 g + s)
    V aw[NB], af[NB];
    const bool has_f = NB == 1 ? !compute : compute;
    {
        const int i = 16 * w + K::arow(c);
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int j = 16 * q + 4 * g + s;
                const bool in = i < n && j < n;
                aw[q][s] = compute && in ? (S)(a.cw * a.W[i * n + j]) : S(0);
                af[q][s] = has_f && in ? (S)(a.cf * a.F[i * n + j]) : S(0);
            }
    }
    auto frag = [&](const S (*X)[XP], const int q, const int b) {
        return *reinterpret_cast<const V*>(&X[16 * b + c][16 * q + 4 * g]);
    };
    // each(q, b, v): block q of column block b as it is read
    auto contract = [&](const V (&m)[NB], const S (*X)[XP], V (&acc)[CB], auto&& each) {
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                const V v = frag(X, q, b);
#pragma unroll
                for (int s = 0; s < 4; ++s) acc[b] = K::mfma(m[q][s], v[s], acc[b]);
                each(q, b, v);
            }
    };
    auto nothing = [](int, int, const V&) {};

    // ---- compute waves: spins of rows i0 .. i0 + 3 of trajectory tl
    const int tl = CB == 1 ? (c & 7) : c, i0 = 16 * w + 4 * g;
    const bool isy = CB == 1 && c >= 8;
    const int64_t k = kb + tl;
    S x[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0}, z[4] = {0, 0, 0, 0};
    auto put = [&](S (*X)[XP], const S (&vx)[4], const S (&vy)[4]) {
        if constexpr (CB == 2) {
            *reinterpret_cast<V*>(&X[c][i0]) = V{vx[0], vx[1], vx[2], vx[3]};
            *reinterpret_cast<V*>(&X[16 + c][i0]) = V{vy[0], vy[1], vy[2], vy[3]};
        } else {
            V v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = isy ? vy[r] : vx[r];
            *reinterpret_cast<V*>(&X[c][i0]) = v;
        }
    };
    auto fields = [&](const V (&acc)[CB], S (&fx)[4], S (&fy)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (CB == 2) {
                fx[r] = acc[0][r];
                fy[r] = acc[1][r];
            } else {
                const S o = ror8(acc[0][r]);
                fx[r] = isy ? o : acc[0][r];
                fy[r] = isy ? acc[0][r] : o;
            }
        }
    };
    // the x and y totals of the lane's trajectory
    auto totals = [&](const ColumnSum<S, NB> (&cs)[CB], S& tx, S& ty) {
        const S v = cs[0].total();
        if constexpr (CB == 2) {
            tx = v;
            ty = cs[1].total();
        } else {
            const S o = ror8(v);
            tx = isy ? o : v;
            ty = isy ? v : o;
        }
    };
    // NB = 1: the wave holds all spins of its trajectories, and sums them while
    // they go through LDS
    auto own_total = [&](const S (&v)[4]) {
        return across32(across16(((v[0] + v[1]) + v[2]) + v[3]));
    };
    S hx[4], hy[4], dx[4], dy[4], dz[4], px[4], py[4], Sx = 0, Sy = 0, gx = 0, gy = 0;
    // predictor: the fields at s_n and its increment.  acc: what the noise
    // gives already (NB = 1, else zero), then the pump and the noise; g0, g1:
    // the collective noise field where acc does not hold it
    auto predictor = [&](V (&acc)[CB], const S (*zb)[XP], const S g0, const S g1) {
        if constexpr (NB == 1) {
            contract(aw, Xs, acc, nothing);
            Sx = own_total(x);
            Sy = own_total(y);
        } else {
            ColumnSum<S, NB> cs[CB];
            contract(aw, Xs, acc, [&](const int q, const int b, const V& v) { cs[b].add(q, v); });
            contract(af, zb, acc, nothing);
            totals(cs, Sx, Sy);
        }
        gx = g0;
        gy = g1;
        const S cx0 = a.c1 * Sx + gx, cy0 = a.c1 * Sy + gy;
        fields(acc, hx, hy);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const S Hx = hx[r] + cx0, Hy = hy[r] + cy0;
            if (a.sib) {
                const S bx = S(0.5) * Hy, by = S(-0.5) * Hx;
                const S cx = by * z[r], cy = -(bx * z[r]), cz = bx * y[r] - by * x[r];
                const S f = S(-2) / (S(1) + bx * bx + by * by);
                dx[r] = f * (cx - by * cz);
                dy[r] = f * (cy + bx * cz);
                dz[r] = f * (cz - (bx * cy - by * cx));
            } else {
                dx[r] = z[r] * Hx;
                dy[r] = z[r] * Hy;
                dz[r] = -(x[r] * Hx + y[r] * Hy);
            }
            px[r] = x[r] + dx[r];
            py[r] = y[r] + dy[r];
        }
        put(Xd, dx, dy);
        if constexpr (NB > 1) put(Xp, px, py);
    };
    // corrector: the pump field moves by that of D (Heun) or D / 2 (midpoint),
    // the collective one is that of the predictor's sums (or the mean of both)
    auto corrector = [&](S* red) {
        V acc[CB] = {};
        S fx[4], fy[4], sx = 0, sy = 0, sz = 0, Px, Py;
        if constexpr (NB == 1) {
            contract(aw, Xd, acc, nothing);
            Px = own_total(px);
            Py = own_total(py);
        } else {
            ColumnSum<S, NB> cs[CB];
            contract(aw, Xd, acc, [&](const int q, const int b, const V&) { cs[b].add(q, frag(Xp, q, b)); });
            totals(cs, Px, Py);
        }
        const S cx0 = a.c1 * (a.sib ? S(0.5) * (Sx + Px) : Px) + gx, cy0 = a.c1 * (a.sib ? S(0.5) * (Sy + Py) : Py) + gy;
        fields(acc, fx, fy);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (a.sib) {
                const S Hx = (hx[r] + S(0.5) * fx[r]) + cx0, Hy = (hy[r] + S(0.5) * fy[r]) + cy0;
                const S bx = S(0.5) * Hy, by = S(-0.5) * Hx;
                const S ax = x[r] - by * z[r], ay = y[r] + bx * z[r], az = z[r] - (bx * y[r] - by * x[r]);
                const S bd = bx * ax + by * ay;
                const S inv = S(1) / (S(1) + bx * bx + by * by);
                x[r] = (ax - by * az + bx * bd) * inv;
                y[r] = (ay + bx * az + by * bd) * inv;
                z[r] = (az - (bx * ay - by * ax)) * inv;
            } else {
                const S Hx = (hx[r] + fx[r]) + cx0, Hy = (hy[r] + fy[r]) + cy0;
                const S px = x[r] + dx[r], py = y[r] + dy[r], pz = z[r] + dz[r];
                const S ex = pz * Hx, ey = pz * Hy, ez = -(px * Hx + py * Hy);
                x[r] = x[r] + S(0.5) * (dx[r] + ex);
                y[r] = y[r] + S(0.5) * (dy[r] + ey);
                z[r] = z[r] + S(0.5) * (dz[r] + ez);
            }
            sx += x[r];
            sy += y[r];
            sz += z[r];
        }
        put(Xs, x, y);
        if constexpr (NB > 1) {
            if (!isy) *reinterpret_cast<V*>(&Xz[tl][i0]) = V{z[0], z[1], z[2], z[3]};
        } else if (!isy) {   // red: [4 (g)][3][T]
            red[(g * 3 + 0) * T + tl] = sx;
            red[(g * 3 + 1) * T + tl] = sy;
            red[(g * 3 + 2) * T + tl] = sz;
        }
    };

    // ---- producer waves
    const int pw = wave - NB, pl = pw * 64 + lane;
    const int ns = (n + 1) / 2;
    // item it of a step's noise: one Philox call of a (trajectory, slot), both
    // pairs in FP32, one pair per item in FP64 (half as long a chain)
    constexpr int HALVES = sizeof(S) == 8 ? 2 : 1;
    const int items = T * ns * HALVES;
    auto pump_item = [&](const int it, const int64_t st, S (&zb)[COLS][XP]) {
        const int q = it / HALVES, h = it % HALVES, t = q / ns, m = q - t * ns;
        const U4 wd = philox4x32_10(U4{(uint32_t)m, (uint32_t)(kb + t), (uint32_t)st, TAG_PUMP | (a.point << 8)}, a.k0,
                                    a.k1);
        const int cx = t, cy = (CB == 1 ? 8 : 16) + t;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (HALVES == 2 && e == 1) break;
            const bool second = HALVES == 2 ? h == 1 : e == 1;
            S za, zc;
            box_muller(second ? wd.z : wd.x, second ? wd.w : wd.y, za, zc);
            const int i = 2 * m + (second ? 1 : 0);
            if (i < n) {
                zb[cx][i] = za;
                zb[cy][i] = zc;
            }
        }
    };
    auto collective_item = [&](const int t, const int64_t st, S (&gb)[T][2]) {
        const U4 wd = philox4x32_10(U4{0u, (uint32_t)(kb + t), (uint32_t)st, TAG_COLLECTIVE | (a.point << 8)}, a.k0,
                                    a.k1);
        S g0, g1;
        box_muller(wd.x, wd.y, g0, g1);
        gb[t][0] = g0;
        gb[t][1] = g1;
    };
    // window moments (first producer wave): lanes t < T keep the Kahan sums of
    // trajectory t
    S msum[5] = {0, 0, 0, 0, 0}, mcmp[5] = {0, 0, 0, 0, 0};
    auto moments = [&](const S Tx, const S Ty, const S Tz) {
        const S T2 = S(0.25) * (Tx * Tx + Ty * Ty);
        const S mv[5] = {T2, T2 * Tz, T2 * T2, Tz, Tz * Tz};
#pragma unroll
        for (int m = 0; m < 5; ++m) kahan(msum[m], mcmp[m], mv[m]);
    };
    // NB = 1, the steps st .. st + nst - 1 of a batch: lane l < 3 T adds the
    // partial sums of component l / T of trajectory l % T
    auto observe = [&](const int64_t st, const int nst, const S (&rb)[U][NB == 1 ? 4 : 1][3][T]) {
        for (int u = 0; u < nst; ++u) {
            if (st + u + 1 <= a.burnin) continue;
            const int l = lane < 3 * T ? lane : 0, cc = l / T, t = l % T;
            const S v = (rb[u][0][cc][t] + rb[u][1][cc][t]) + (rb[u][2][cc][t] + rb[u][3][cc][t]);
            moments(v, __shfl(v, T + (lane % T)), __shfl(v, 2 * T + (lane % T)));
        }
    };
    // NB > 1: the state after step st, from the columns
    auto observe_columns = [&](const int64_t st) {
        if (st + 1 <= a.burnin) return;
        ColumnSum<S, NB> cs[CB], cz;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
#pragma unroll
            for (int b = 0; b < CB; ++b) cs[b].add(q, frag(Xs, q, b));
            cz.add(q, *reinterpret_cast<const V*>(&Xz[tl][16 * q + 4 * g]));
        }
        S Tx, Ty;
        totals(cs, Tx, Ty);
        moments(Tx, Ty, cz.total());
    };

    if (compute) {
        if (k < a.B)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + r < n) {
                    x[r] = a.s_in[k * a.P + i0 + r];
                    y[r] = a.s_in[SP + k * a.P + i0 + r];
                    z[r] = a.s_in[2 * SP + k * a.P + i0 + r];
                }
        put(Xs, x, y);
    }
    __syncthreads();   // Z cleared, Xs written

    const S c2 = a.c2;
    if constexpr (NB == 1) {
        // noise fields of the steps st .. st + nst - 1, one producer wave per step
        auto produce = [&](const int64_t st, const int nst, const int buf) {
            for (int u = pw; u < nst; u += PRODUCERS) {
                for (int it = lane; it < items; it += 64) pump_item(it, st + u, Z[pw]);
                if (lane < T) collective_item(lane, st + u, Gn[pw]);
                wave_lds_fence();
                V acc[CB] = {};
                contract(af, Z[pw], acc, nothing);
                S fx[4], fy[4];
                fields(acc, fx, fy);
                const S qx = c2 * Gn[pw][tl][0], qy = c2 * Gn[pw][tl][1];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    fx[r] += qx;
                    fy[r] += qy;
                }
                if constexpr (CB == 2) {
                    *reinterpret_cast<V*>(&Q[buf * U + u][c][4 * g]) = V{fx[0], fx[1], fx[2], fx[3]};
                    *reinterpret_cast<V*>(&Q[buf * U + u][16 + c][4 * g]) = V{fy[0], fy[1], fy[2], fy[3]};
                } else {
                    V v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = isy ? fy[r] : fx[r];
                    *reinterpret_cast<V*>(&Q[buf * U + u][c][4 * g]) = v;
                }
                wave_lds_fence();
            }
        };
        auto len = [&](const int64_t st) { return (int)(a.n_steps - st < U ? a.n_steps - st : U); };
        if (!compute && a.n_steps > 0) produce(0, len(0), 0);
        __syncthreads();
        int buf = 0;
        for (int64_t st = 0; st < a.n_steps; st += U, buf ^= 1) {
            const int nst = len(st);
            if (compute) {
                for (int u = 0; u < nst; ++u) {
                    V acc[CB];
#pragma unroll
                    for (int b = 0; b < CB; ++b)
                        acc[b] = *reinterpret_cast<const V*>(&Q[buf * U + u][16 * b + c][4 * g]);
                    predictor(acc, nullptr, S(0), S(0));
                    wave_lds_fence();
                    corrector(&R[buf][u][0][0][0]);
                    wave_lds_fence();
                }
            } else {
                if (st + nst < a.n_steps) produce(st + nst, len(st + nst), buf ^ 1);
                if (pw == 0 && st > 0) observe(st - U, U, R[buf ^ 1]);
            }
            __syncthreads();
        }
        if (!compute && pw == 0 && a.n_steps > 0) {
            const int64_t last = (a.n_steps - 1) / U * U;
            observe(last, len(last), R[buf ^ 1]);
        }
    } else {
        // items [0, cut) of a step are drawn while the predictor runs (two
        // thirds of its time), the rest while the corrector does
        const int all = items + T, cut = (2 * all / 3 + 255) / 256 * 256;
        auto produce = [&](const int from, const int to, const int64_t st, const int buf) {
            for (int it = from + pl; it < to; it += 64 * PRODUCERS) {
                if (it < items) pump_item(it, st, Z[buf]);
                else collective_item(it - items, st, Gn[buf]);
            }
        };
        if (!compute && a.n_steps > 0) produce(0, all, 0, 0);
        __syncthreads();
        int buf = 0;
        for (int64_t st = 0; st < a.n_steps; ++st, buf ^= 1) {
            if (compute) {
                V acc[CB] = {};
                predictor(acc, Z[buf], c2 * Gn[buf][tl][0], c2 * Gn[buf][tl][1]);
            } else {
                if (pw == 0 && st > 0) observe_columns(st - 1);
                if (st + 1 < a.n_steps) produce(0, min(cut, all), st + 1, buf ^ 1);
            }
            __syncthreads();
            if (compute) corrector(nullptr);
            else if (st + 1 < a.n_steps) produce(min(cut, all), all, st + 1, buf ^ 1);
            __syncthreads();
        }
        if (!compute && pw == 0 && a.n_steps > 0) observe_columns(a.n_steps - 1);
    }

    if (compute) {
        if (k < a.B && !isy)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (i0 + r < n) {
                    a.s_out[k * a.P + i0 + r] = x[r];
                    a.s_out[SP + k * a.P + i0 + r] = y[r];
                    a.s_out[2 * SP + k * a.P + i0 + r] = z[r];
                }
    } else if (pw == 0 && lane < T && kb + lane < a.B) {
#pragma unroll
        for (int m = 0; m < 5; ++m) {
            a.mom[(2 * m) * a.Bp + kb + lane] = msum[m];
            a.mom[(2 * m + 1) * a.Bp + kb + lane] = mcmp[m];
        }
    }
}

// midpoint rotation of the semi-implicit scheme (same closed form as the step kernels)
template <typename S>
__device__ __forceinline__ void rotate(S x, S y, S z, S Hx, S Hy, S& ox, S& oy, S& oz) {
    const S bx = S(0.5) * Hy, by = S(-0.5) * Hx;
    const S ax = x - by * z, ay = y + bx * z, az = z - (bx * y - by * x);
    const S bd = bx * ax + by * ay;
    const S inv = S(1) / (S(1) + bx * bx + by * by);
    ox = (ax - by * az + bx * bd) * inv;
    oy = (ay + bx * az + by * bd) * inv;
    oz = (az - (bx * ay - by * ax)) * inv;
}

// The shortest chains, a spin to a lane: a trajectory occupies NL = 2^k >= N
// lanes of one wave and forms its products from rows of the operands and the
// spin vectors in LDS.  No lane works on padding, where the matrix kernel above
// pads to 16 spins, so it is the faster one for few spins and many trajectories
// (see lanes_apply).  Bound by the LDS reads of its products.
template <typename S, int NL>
__global__ __launch_bounds__(LANES_THREADS) void lanes_run_kernel(SmallArgs<S> a) {
    constexpr int TPB = LANES_THREADS / NL;            // trajectories per block
    __shared__ S Aw[NL * NL];                          // -dt/2 W, row-major N x N
    __shared__ S Af[NL * NL];                          // -sqrt(dt) F
    __shared__ S vx[TPB][NL], vy[TPB][NL], ux[TPB][NL], uy[TPB][NL];
    const int n = a.n;
    const int64_t B = a.B, P = a.P, Bp = a.Bp;
    const uint32_t k0 = a.k0, k1 = a.k1, point = a.point;
    const S c1 = a.c1, c2 = a.c2;
    for (int t = threadIdx.x; t < n * n; t += LANES_THREADS) {
        Aw[t] = (S)(a.cw * a.W[t]);
        Af[t] = (S)(a.cf * a.F[t]);
    }
    const int tl = threadIdx.x / NL, i = threadIdx.x % NL;   // trajectory in block, spin
    const int64_t k = (int64_t)blockIdx.x * TPB + tl;
    const bool live = k < B && i < n;
    const int64_t SP = Bp * P;
    S x = 0, y = 0, z = 0;
    if (live) {
        x = a.s_in[k * P + i];
        y = a.s_in[SP + k * P + i];
        z = a.s_in[2 * SP + k * P + i];
    }
    S msum[5] = {0, 0, 0, 0, 0}, mcmp[5] = {0, 0, 0, 0, 0};
    const S* aw = Aw + i * n;
    const S* af = Af + i * n;
    __syncthreads();

    for (int64_t st = 0; st < a.n_steps; ++st) {
        // noise of the step (counters of the multi-kernel path)
        S zx = 0, zy = 0, g0 = 0, g1 = 0;
        {
            const uint32_t ks = (uint32_t)k, ns = (uint32_t)st;
            const U4 w = philox4x32_10(U4{(uint32_t)(i >> 1), ks, ns, TAG_PUMP | (point << 8)}, k0, k1);
            S a0, a1, a2, a3;
            box_muller(w.x, w.y, a0, a1);
            box_muller(w.z, w.w, a2, a3);
            if (live) {
                zx = (i & 1) ? a2 : a0;
                zy = (i & 1) ? a3 : a1;
            }
            const U4 v = philox4x32_10(U4{0u, ks, ns, TAG_COLLECTIVE | (point << 8)}, k0, k1);
            box_muller(v.x, v.y, g0, g1);
        }
        // stage 1: fields at s_n
        vx[tl][i] = x;
        vy[tl][i] = y;
        ux[tl][i] = zx;
        uy[tl][i] = zy;
        __syncthreads();
        S Yx = 0, Yy = 0, Qx = 0, Qy = 0, Sx = 0, Sy = 0;
        for (int j = 0; j < n; ++j) {
            Yx += aw[j] * vx[tl][j];
            Yy += aw[j] * vy[tl][j];
            Qx += af[j] * ux[tl][j];
            Qy += af[j] * uy[tl][j];
            Sx += vx[tl][j];
            Sy += vy[tl][j];
        }
        const S Hx = (Yx + Qx) + (c1 * Sx + c2 * g0), Hy = (Yy + Qy) + (c1 * Sy + c2 * g1);
        S px, py, pz, dx = 0, dy = 0, dz = 0;
        if (a.sib) {
            rotate(x, y, z, Hx, Hy, px, py, pz);
        } else {
            dx = z * Hx;
            dy = z * Hy;
            dz = -(x * Hx + y * Hy);
            px = x + dx;
            py = y + dy;
            pz = z + dz;
        }
        if (!live) px = py = pz = 0;
        // stage 2: fields at the predictor (Heun) or the midpoint (semi-implicit)
        const S mx = a.sib ? S(0.5) * (x + px) : px, my = a.sib ? S(0.5) * (y + py) : py;
        __syncthreads();   // stage-1 reads done
        vx[tl][i] = mx;
        vy[tl][i] = my;
        __syncthreads();
        S Y2x = 0, Y2y = 0, S2x = 0, S2y = 0;
        for (int j = 0; j < n; ++j) {
            Y2x += aw[j] * vx[tl][j];
            Y2y += aw[j] * vy[tl][j];
            S2x += vx[tl][j];
            S2y += vy[tl][j];
        }
        const S H2x = (Y2x + Qx) + (c1 * S2x + c2 * g0), H2y = (Y2y + Qy) + (c1 * S2y + c2 * g1);
        if (a.sib) {
            rotate(x, y, z, H2x, H2y, x, y, z);
        } else {
            const S ex = pz * H2x, ey = pz * H2y, ez = -(px * H2x + py * H2y);
            x = x + S(0.5) * (dx + ex);
            y = y + S(0.5) * (dy + ey);
            z = z + S(0.5) * (dz + ez);
        }
        if (!live) x = y = z = 0;
        // window moments of the new state
        if (st + 1 > a.burnin) {
            __syncthreads();   // stage-2 reads done
            vx[tl][i] = x;
            vy[tl][i] = y;
            ux[tl][i] = z;
            __syncthreads();
            if (i == 0) {
                S Tx = 0, Ty = 0, Tz = 0;
                for (int j = 0; j < n; ++j) {
                    Tx += vx[tl][j];
                    Ty += vy[tl][j];
                    Tz += ux[tl][j];
                }
                const S T2 = S(0.25) * (Tx * Tx + Ty * Ty);
                const S v[5] = {T2, T2 * Tz, T2 * T2, Tz, Tz * Tz};
#pragma unroll
                for (int m = 0; m < 5; ++m) kahan(msum[m], mcmp[m], v[m]);
            }
        }
        __syncthreads();   // all reads of this step done before the next step's writes
    }
    if (k < B) {
        if (i < n) {
            a.s_out[k * P + i] = x;
            a.s_out[SP + k * P + i] = y;
            a.s_out[2 * SP + k * P + i] = z;
        }
        if (i == 0)
#pragma unroll
            for (int m = 0; m < 5; ++m) {
                a.mom[(2 * m) * Bp + k] = msum[m];
                a.mom[(2 * m + 1) * Bp + k] = mcmp[m];
            }
    }
}

template <typename S, int NB, int CB>
int launch_small_t(const SmallArgs<S>& a, hipStream_t st) {
    constexpr int T = 8 * CB;
    hipLaunchKernelGGL((small_run_kernel<S, NB, CB>), dim3((unsigned)((a.B + T - 1) / T)),
                       dim3(64 * (NB + PRODUCERS)), 0, st, a);
    TWA_HIP_CHECK(hipGetLastError());
    return TWA_OK;
}

template <typename S, int NB>
int launch_small_nb(const SmallArgs<S>& a, int nb, int cb, hipStream_t st) {
    if constexpr (NB > Small<S>::MAX_NB) {
        set_error("fused small-N path: too many atoms");
        return TWA_EINVAL;
    } else {
        if (nb > NB) return launch_small_nb<S, NB + 1>(a, nb, cb, st);
        return cb == 1 ? launch_small_t<S, NB, 1>(a, st) : launch_small_t<S, NB, 2>(a, st);
    }
}

template <typename S, int NL>
int launch_lanes_t(const SmallArgs<S>& a, hipStream_t st) {
    constexpr int TPB = LANES_THREADS / NL;
    hipLaunchKernelGGL((lanes_run_kernel<S, NL>), dim3((unsigned)((a.B + TPB - 1) / TPB)), dim3(LANES_THREADS), 0, st, a);
    TWA_HIP_CHECK(hipGetLastError());
    return TWA_OK;
}

// Where a spin to a lane is faster, in us a step against the matrix kernel.
// FP32: to N = 4 everywhere (N = 2 1.3 against 1.5 at 4096 trajectories, 8.5
// against 48 at 131072), and past the 4096 trajectories that the matrix kernel
// takes in one round, to N = 15 (8192: N = 8 1.6 against 3.0, N = 15 2.7 against
// 3.1; N = 16, its rows on the same LDS banks, 4.0 against 3.1) and to N = 27
// where N is no multiple of 4 (32768: N = 17 14.6 against 18.7, N = 27 19.0
// against 18.9, N = 20 21.8 against 18.9).  FP64: past 4096 to N = 8 (8192: 3.5
// against 4.0, N = 9 5.0 against 4.1).
template <typename S>
bool lanes_apply(int n, int64_t B) {
    if (sizeof(S) == 8) return n <= 8 && B > 4096;
    return n <= 4 || (B > 4096 && (n <= 15 || (n <= 27 && n % 4 != 0)));
}

template <typename S>
int launch_small_s(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, const twa_pump* pump, double dt,
                   int64_t n_steps, int out_cur, hipStream_t st) {
    SmallArgs<S> a{};
    a.n = (int)g.N;
    a.B = g.B;
    a.P = g.P;
    a.Bp = g.Bp;
    a.W = pump->W;
    a.F = pump->F;
    a.cw = -0.5 * dt;
    a.cf = -std::sqrt(dt);
    a.c1 = (S)c.c1;
    a.c2 = (S)c.c2;
    a.k0 = c.key0;
    a.k1 = c.key1;
    a.point = (uint32_t)c.point;
    a.n_steps = n_steps;
    a.burnin = c.burnin;
    a.sib = g.integrator == TWA_INT_SIB ? 1 : 0;
    a.s_in = static_cast<const S*>(b.s[0]);
    a.s_out = static_cast<S*>(b.s[out_cur]);
    a.mom = static_cast<S*>(b.mom);
    if (lanes_apply<S>(a.n, a.B)) {
        if (a.n <= 8) return launch_lanes_t<S, 8>(a, st);
        if constexpr (sizeof(S) == 4) return a.n <= 16 ? launch_lanes_t<S, 16>(a, st) : launch_lanes_t<S, 32>(a, st);
    }
    // 8 trajectories per workgroup up to one workgroup per compute unit (us a step: FP64 N = 50 x 512 4.5 against
    // 7.0 with 16, FP32 N = 100 x 2000 5.2 against 7.9), then 16 (FP32 N = 128 x 4096 9.1 against 11.1)
    const int cb = g.B <= 8 * 256 ? 1 : 2;
    return launch_small_nb<S, 1>(a, (int)((g.N + 15) / 16), cb, st);
}

}  // namespace

bool small_path_applies(int precision, int64_t N, int64_t n_lags) {
    if (n_lags != 0) return false;
    if (precision == TWA_PREC_FP64) return N <= 16 * Small<double>::MAX_NB;
    return precision == TWA_PREC_FP32 && N <= 16 * Small<float>::MAX_NB;
}

int launch_small_run(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, const twa_pump* pump,
                     double dt, int64_t n_steps, int out_cur, hipStream_t st) {
    if (!small_path_applies(g.precision, g.N, 0)) {
        set_error("fused small-N path: FP64 with N <= 64 or FP32 with N <= 128 only");
        return TWA_EINVAL;
    }
    if (g.precision == TWA_PREC_FP64) return launch_small_s<double>(g, b, c, pump, dt, n_steps, out_cur, st);
    return launch_small_s<float>(g, b, c, pump, dt, n_steps, out_cur, st);
}

}  // namespace twa
