// Run driver of the C ABI: buffer management, the step loop (direct launches
// or replayed hipGraphs), and the host-side finalisation of the few kB of
// accumulators copied back once at the end (the paper's End Matter advises a
// single device-to-host transfer at the end of the simulation).
#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstring>
#include <vector>

#include "twa_internal.h"
#include "twa_run.h"

namespace twa {

static thread_local std::string g_err;

std::recursive_mutex& api_mutex() {
    static std::recursive_mutex m;
    return m;
}
void set_error(const std::string& msg) { g_err = msg; }

int gemm_elt_bytes(int precision) {
    switch (precision) {
        case TWA_PREC_FP64: return 8;
        case TWA_PREC_FP32: return 4;
        default: return 2;
    }
}
int state_elt_bytes(int precision) { return precision == TWA_PREC_FP64 ? 8 : 4; }
int operand_split(int precision) { return precision == TWA_PREC_BF16X3 ? 2 : 1; }

static int n_compute_units() {
    static int ncu = 0;
    if (ncu <= 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
            ncu = 256;
    }
    return ncu;
}

// Tile shape of a contraction.  In FP64 the smallest tiles that fill the
// device: bound by its MFMA, it takes 16x32, one wave each, up to one to a SIMD
// (600 x 400, 950 of them, 65 against 89 us with 64x64; 700 x 512, 1408, 125
// against 98), then 32x32 up to three to a unit (700 x 512 86 us, 1500 x 256
// 164 against 191; 1000 x 512, four, 194 against 136), then 64x64, its waves in
// two groups over K where each has a compute unit to itself and the
// contraction is long enough to pay for adding the sums (500 x 1000 84 against
// 81 us, 1000 x 512 130 against 136).
// The other precisions: the rows of a tile follow from N (16 to N = 48, 64 to
// N = 768), above that 128 or 320, whichever gives the shorter estimate of
// rounds of tiles x work per tile / rate per tile (the 320x256 tile moves 45 %
// fewer bytes per flop than 128x128, whose bound that is, and runs 1.64 times
// faster, but needs enough tiles to fill the device).  The rows set the order
// in which a trajectory's spins are summed, so they follow from this rule
// alone.  The columns show in no result: narrower tiles where the wide ones are
// too few to fill the device.  64x32 to one a compute unit (FP32 us a step at
// 201 x 500 25.6 against 26.4 with 64x64, at 600 x 400 46.4 against 47.5; past
// that two share a unit's SIMDs unevenly, 400 x 600 54.4 against 36.8).  128x64
// in FP32 throughout (1000 x 1024 123 against 215 with 128x128, 1000 x 4096 394
// against 440, 2000 x 2048 751 against 817), in split BF16 to one a unit
// (2000 x 512 136 against 165; 4096 x 512, two, 334 against 318), in BF16 to two
// (2000 x 512 54 against 75, 4096 x 512 124 against 132; 4096 x 1024, four, 282
// against 254).
int pick_tile_cfg(int precision, int64_t N, int64_t n_traj) {
    const int64_t ncu = n_compute_units();
    auto tiles = [&](int cfg) {
        const TileCfg& t = tile_cfg(precision, cfg);
        return (round_up(N, t.mt) / t.mt) * (2 * round_up(n_traj, t.nt / 2) / t.nt);
    };
    if (precision == TWA_PREC_FP64) {
        if (N <= 48 || tiles(0) <= 4 * ncu) return 0;
        return tiles(9) <= 3 * ncu ? 9 : tiles(1) <= ncu && N >= 600 ? 10 : 1;
    }
    auto est = [&](int cfg, double rate) {
        const TileCfg& t = tile_cfg(precision, cfg);
        return (double)((tiles(cfg) + ncu - 1) / ncu) * (double)(t.mt * t.nt) / rate;
    };
    if (N <= 48) return 0;
    if (N <= 768) return tiles(9) <= ncu ? 9 : 1;
    if (est(7, 1.64) < est(2, 1.0)) return 7;
    if (precision == TWA_PREC_FP32) return 10;
    if (operand_split(precision) > 1) return tiles(10) <= ncu ? 10 : 2;
    return tiles(10) <= 2 * ncu ? 10 : 3;
}

// ---------------------------------------------------------------------------
// host finalisation
void finalize_moments(const std::vector<double>& traj, int64_t B, twa_observables* o) {
    // traj: [B][5] per-trajectory window averages
    const int J = (int)std::min<int64_t>(32, B);
    double bsum[32 * 5] = {0}, bcnt[32] = {0};
    for (int64_t k = 0; k < B; ++k) {
        const int j = (int)((k * J) / B);
        for (int m = 0; m < 5; ++m) bsum[(size_t)j * 5 + m] += traj[(size_t)k * 5 + m];
        bcnt[(size_t)j] += 1.0;
    }
    finalize_blocks(bsum, bcnt, J, B, o);
}

void finalize_blocks(const double* bsum, const double* bcnt, int J, int64_t B, twa_observables* o) {
    double tot[5] = {0, 0, 0, 0, 0};
    for (int j = 0; j < J; ++j)
        for (int m = 0; m < 5; ++m) tot[m] += bsum[(size_t)j * 5 + m];
    auto derive = [](const double* m, double* d) {
        const double T2 = m[0], T3 = m[1], T4 = m[2], Z = m[3], ZZ = m[4];
        const double spsm = T2 + 0.5 * Z;
        const double num = T4 + 2.0 * T3 - Z / 3.0 + 0.5 * ZZ - (4.0 / 3.0) * T2;
        d[0] = Z;
        d[1] = spsm;
        d[2] = num / (spsm * spsm);
    };
    double mean[8];
    for (int m = 0; m < 5; ++m) mean[m] = tot[m] / (double)B;
    derive(mean, mean + 5);
    double se[8];
    if (J >= 2) {
        double vals[32 * 8];
        for (int j = 0; j < J; ++j) {
            double* v = &vals[(size_t)j * 8];
            for (int m = 0; m < 5; ++m) v[m] = (tot[m] - bsum[(size_t)j * 5 + m]) / ((double)B - bcnt[(size_t)j]);
            derive(v, v + 5);
        }
        for (int c = 0; c < 8; ++c) {
            double mu = 0;
            for (int j = 0; j < J; ++j) mu += vals[(size_t)j * 8 + c];
            mu /= J;
            double ss = 0;
            for (int j = 0; j < J; ++j) {
                const double d = vals[(size_t)j * 8 + c] - mu;
                ss += d * d;
            }
            se[c] = std::sqrt((double)(J - 1) / J * ss);
        }
    } else {
        for (int c = 0; c < 8; ++c) se[c] = NAN;
    }
    o->T2 = mean[0]; o->T3 = mean[1]; o->T4 = mean[2]; o->Z = mean[3]; o->ZZ = mean[4];
    o->Sz = mean[5]; o->SpSm = mean[6]; o->g2 = mean[7];
    o->T2_se = se[0]; o->T3_se = se[1]; o->T4_se = se[2]; o->Z_se = se[3]; o->ZZ_se = se[4];
    o->Sz_se = se[5]; o->SpSm_se = se[6]; o->g2_se = se[7];
}

void finalize_decay(const std::vector<double>& traj, int64_t B, twa_observables* o) {
    // traj: [B][9] per-trajectory window averages of (E2, E2^2, E2 D, Q3, R, D^2, U, V, D);
    // intensity I = E2 + D/2 and the four-point function of SM Sec. S1 step 6, g2 = four-point / I^2
    const int J = (int)std::min<int64_t>(32, B);
    std::vector<double> bsum((size_t)J * 9, 0.0), bcnt((size_t)J, 0.0);
    for (int64_t k = 0; k < B; ++k) {
        const int j = (int)((k * J) / B);
        for (int m = 0; m < 9; ++m) bsum[(size_t)j * 9 + m] += traj[(size_t)k * 9 + m];
        bcnt[(size_t)j] += 1.0;
    }
    double tot[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int j = 0; j < J; ++j)
        for (int m = 0; m < 9; ++m) tot[m] += bsum[(size_t)j * 9 + m];
    auto derive = [](const double* m, double* d) {
        const double E2 = m[0], E2E2 = m[1], E2D = m[2], Q3 = m[3], R = m[4], DD = m[5], U = m[6], V = m[7], D = m[8];
        const double inten = E2 + 0.5 * D;
        const double num = E2E2 + E2D + Q3 - R / 3.0 + 0.25 * (DD + U) - (4.0 / 3.0) * V;
        d[0] = inten;
        d[1] = num / (inten * inten);
    };
    double mean[9], dm[2];
    for (int m = 0; m < 9; ++m) mean[m] = tot[m] / (double)B;
    derive(mean, dm);
    o->I_gen = dm[0];
    o->g2_gen = dm[1];
    o->I_gen_se = o->g2_gen_se = NAN;
    if (J >= 2) {
        std::vector<double> vals((size_t)J * 2);
        for (int j = 0; j < J; ++j) {
            double v[9];
            for (int m = 0; m < 9; ++m) v[m] = (tot[m] - bsum[(size_t)j * 9 + m]) / ((double)B - bcnt[(size_t)j]);
            derive(v, &vals[(size_t)j * 2]);
        }
        double se[2];
        for (int c = 0; c < 2; ++c) {
            double mu = 0;
            for (int j = 0; j < J; ++j) mu += vals[(size_t)j * 2 + c];
            mu /= J;
            double ss = 0;
            for (int j = 0; j < J; ++j) {
                const double d = vals[(size_t)j * 2 + c] - mu;
                ss += d * d;
            }
            se[c] = std::sqrt((double)(J - 1) / J * ss);
        }
        o->I_gen_se = se[0];
        o->g2_gen_se = se[1];
    }
}

// iterative radix-2 FFT computing sum_l c_l e^{+2 pi i k l / n}
static void fft_pos(std::vector<std::complex<double>>& a) {
    const size_t n = a.size();
    for (size_t i = 1, j = 0; i < n; ++i) {
        size_t bit = n >> 1;
        for (; j & bit; bit >>= 1) j ^= bit;
        j ^= bit;
        if (i < j) std::swap(a[i], a[j]);
    }
    for (size_t len = 2; len <= n; len <<= 1) {
        const double ang = 2.0 * M_PI / (double)len;
        const std::complex<double> wl(std::cos(ang), std::sin(ang));
        for (size_t i = 0; i < n; i += len) {
            std::complex<double> w(1.0, 0.0);
            for (size_t j = 0; j < len / 2; ++j) {
                const std::complex<double> u = a[i + j], v = a[i + j + len / 2] * w;
                a[i + j] = u + v;
                a[i + j + len / 2] = u - v;
                w *= wl;
            }
        }
    }
}

// S(omega_k) = 2 tau Re sum_l c_l e^{i omega_k l tau}, trapezoid weights at the
// ends, omega_k = 2 pi k / (n tau) with n = 8 L; FWHM around the global peak.
double linewidth_of(const std::vector<std::complex<double>>& corr, double tau) {
    const size_t L = corr.size();
    if (L < 2) return NAN;
    const size_t n = 8 * L;
    std::vector<std::complex<double>> c(n, 0.0);
    for (size_t l = 0; l < L; ++l) c[l] = corr[l];
    c[0] *= 0.5;
    c[L - 1] *= 0.5;
    std::vector<double> S(n);
    if ((n & (n - 1)) == 0) {
        fft_pos(c);
        for (size_t k = 0; k < n; ++k) S[k] = 2.0 * tau * c[k].real();
    } else {
        for (size_t k = 0; k < n; ++k) {
            double acc = 0;
            for (size_t l = 0; l < L; ++l) {
                const double ph = 2.0 * M_PI * (double)((k * l) % n) / (double)n;
                acc += c[l].real() * std::cos(ph) - c[l].imag() * std::sin(ph);
            }
            S[k] = 2.0 * tau * acc;
        }
    }
    // reorder to ascending omega: k = n/2 .. n-1 are negative frequencies
    std::vector<double> om(n), Sp(n);
    const size_t half = n / 2;
    for (size_t q = 0; q < n; ++q) {
        const size_t k = (q + half + (n % 2)) % n;   // matches fftfreq ordering after argsort
        const long kk = (k < (n + 1) / 2) ? (long)k : (long)k - (long)n;
        om[q] = 2.0 * M_PI * (double)kk / ((double)n * tau);
        Sp[q] = S[k];
    }
    size_t kp = 0;
    for (size_t q = 1; q < n; ++q)
        if (Sp[q] > Sp[kp]) kp = q;
    const double hm = 0.5 * Sp[kp];
    size_t i = kp;
    while (i > 0 && Sp[i] > hm) --i;
    if (Sp[i] > hm) return NAN;
    const double left = om[i] + (hm - Sp[i]) * (om[i + 1] - om[i]) / (Sp[i + 1] - Sp[i]);
    size_t j = kp;
    while (j < n - 1 && Sp[j] > hm) ++j;
    if (Sp[j] > hm) return NAN;
    const double right = om[j - 1] + (hm - Sp[j - 1]) * (om[j] - om[j - 1]) / (Sp[j] - Sp[j - 1]);
    return right - left;
}

int run_status(const char* who, bool nan, double max_norm_dev, double norm_tol) {
    const double tol = effective_norm_tol(norm_tol);
    if (nan) {
        set_error(std::string(who) + ": non-finite values in the state or accumulators");
        return TWA_EUNSTABLE;
    }
    if (tol > 0 && !(max_norm_dev <= tol)) {
        char buf[192];
        std::snprintf(buf, sizeof(buf),
                      "%s: a spin length drifted by %.3g (max_norm_dev) > norm_tol %.3g; Eq. (S1) conserves "
                      "|s_i|^2 -- reduce dt or use the semi-implicit integrator",
                      who, max_norm_dev, tol);
        set_error(buf);
        return TWA_EUNSTABLE;
    }
    return TWA_OK;
}

void finalize_lags(const std::vector<double>& hlag, int64_t L, int J, int64_t B, int64_t stride, double dt,
                   double kappa, twa_observables* out, const twa_outputs* outs) {
    std::vector<std::complex<double>> corr((size_t)L), csym((size_t)L);
    for (int64_t l = 0; l < L; ++l) {
        double s[6] = {0, 0, 0, 0, 0, 0};
        for (int j = 0; j < J; ++j)
            for (int q = 0; q < 6; ++q) s[q] += hlag[((size_t)l * J + j) * 6 + q];
        for (int q = 0; q < 6; ++q) s[q] /= (double)B;
        const std::complex<double> cs(s[0], s[1]);
        // kappa * i * (xx + yy + i yx - i xy)
        const std::complex<double> resp(s[2] + s[5], s[3] - s[4]);
        csym[(size_t)l] = cs;
        corr[(size_t)l] = cs + std::complex<double>(0.0, kappa) * resp;
    }
    const double tau = (double)stride * dt;
    out->linewidth = linewidth_of(corr, tau);
    out->linewidth_sym = linewidth_of(csym, tau);
    if (outs && outs->corr_blocks)
        for (size_t q = 0; q < (size_t)L * J; ++q) {
            outs->corr_blocks[2 * q] = hlag[6 * q];
            outs->corr_blocks[2 * q + 1] = hlag[6 * q + 1];
        }
    if (outs && outs->chi_blocks)
        for (size_t q = 0; q < (size_t)L * J; ++q)
            for (int r = 0; r < 4; ++r) outs->chi_blocks[4 * q + r] = hlag[6 * q + 2 + r];
}

// ---------------------------------------------------------------------------
// the block kept between calls (see Arena)
static struct {
    void* p = nullptr;
    size_t bytes = 0;
    int device = -1;
    bool lent = false;
    int64_t pumps = 0;
} g_kept;

void kept_block_free() {
    if (g_kept.p && !g_kept.lent) {
        hipFree(g_kept.p);
        g_kept.p = nullptr;
        g_kept.bytes = 0;
    }
}
size_t kept_block_bytes() { return g_kept.lent ? 0 : g_kept.bytes; }
void pump_born() { ++g_kept.pumps; }
void pump_gone() {
    if (--g_kept.pumps == 0) kept_block_free();
}

hipError_t device_malloc(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess && g_kept.p && !g_kept.lent) {
        hipGetLastError();
        kept_block_free();
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) *p = nullptr;
    return e;
}

int Arena::commit(bool keep, hipStream_t st) {
    auto padded = [](size_t n) { return (std::max<size_t>(n, 16) + 255) / 256 * 256; };
    size_t zeroed = 0, total = 0;
    for (const Item& it : items_) {
        if (it.zero) zeroed += padded(it.bytes);
        total += padded(it.bytes);
    }
    int dev = 0;
    TWA_HIP_CHECK(hipGetDevice(&dev));
    const bool fits = g_kept.bytes >= total && g_kept.bytes <= std::max<size_t>(8 * total, 16u << 20);
    if (keep && g_kept.p && !g_kept.lent && g_kept.device == dev && fits) {
        block_ = g_kept.p;
        bytes_ = g_kept.bytes;
        g_kept.lent = true;
    } else {
        if (keep) kept_block_free();
        if (device_malloc(&block_, total) != hipSuccess) {
            hipGetLastError();
            set_error("device allocation of " + std::to_string(total) + " bytes failed");
            return TWA_ENOMEM;
        }
        bytes_ = total;
    }
    keep_ = keep;
    char* z = static_cast<char*>(block_);
    char* q = z + zeroed;
    for (const Item& it : items_) {
        char*& at = it.zero ? z : q;
        *it.p = at;
        at += padded(it.bytes);
    }
    // cleared on the call's stream (never the null stream: a null-stream
    // operation would synchronise with streams that other threads may be
    // capturing into graphs)
    if (zeroed) TWA_HIP_CHECK(hipMemsetAsync(block_, 0, zeroed, st));
    return TWA_OK;
}

void Arena::release() {
    if (!block_) return;
    if (g_kept.p == block_) {
        g_kept.lent = false;
    } else if (keep_ && !g_kept.p && g_kept.pumps > 0) {
        size_t freeb = 0, totb = 0;
        int dev = 0;
        if (hipMemGetInfo(&freeb, &totb) == hipSuccess && hipGetDevice(&dev) == hipSuccess && bytes_ <= totb / 64) {
            g_kept.p = block_;
            g_kept.bytes = bytes_;
            g_kept.device = dev;
            g_kept.lent = false;
        } else {
            hipFree(block_);
        }
    } else {
        hipFree(block_);
    }
    block_ = nullptr;
}

void* Arena::detach() {
    void* p = block_;
    block_ = nullptr;
    return p;
}

void add_buffers(const Geometry& g, bool tangents, int64_t L, int J, bool contraction, EnsembleBuffers& b, Arena& ar) {
    const size_t ge = (size_t)gemm_elt_bytes(g.precision), se = (size_t)state_elt_bytes(g.precision);
    const size_t P = (size_t)g.P, Bp = (size_t)g.Bp, C2 = (size_t)g.C2, nmt = (size_t)g.nmt;
    const size_t op = ge * (size_t)operand_split(g.precision);   // bytes per operand value
    const size_t ck = g.coh ? 1 : 0;                              // coherent exchange: one more K block
    // zero at the start: what a run reads before it writes all of (padding of
    // the noise columns, normals of padding trajectories, sums, counters)
    ar.add(b.g, 4 * Bp * se, true);
    ar.add(b.mom, 10 * Bp * se, true);
    ar.add(b.step, 2 * sizeof(int64_t), true);
    ar.add(b.diag, 2 * 1024 * sizeof(float), true);
    ar.add(b.sm0, 2 * Bp * se, true);
    if (L > 0) ar.add(b.lag, (size_t)L * J * 6 * sizeof(double), true);
    ar.add(b.s[0], 3 * Bp * P * se, false);
    ar.add(b.s[1], 3 * Bp * P * se, false);
    ar.add(b.Y, 2 * Bp * P * se, false);
    ar.add(b.norm0, Bp * P * se, false);
    if (contraction) {
        ar.add(b.Xop, C2 * (2 + ck) * P * op, true);
        ar.add(b.Sn, 2 * Bp * se, true);
        ar.add(b.part[0], 3 * nmt * Bp * se, true);
        ar.add(b.part[1], 3 * nmt * Bp * se, true);
        ar.add(b.A, P * (2 + ck) * P * op, false);
        ar.add(b.Dop, C2 * (1 + ck) * P * op, false);
        if (ck) ar.add(b.A2, P * 2 * P * op, false);
        ar.add(b.dlt, 3 * Bp * P * se, false);
    }
    if (tangents) {
        ar.add(b.tXop, 2 * C2 * P * op, true);
        ar.add(b.ts[0], 2 * 3 * Bp * P * se, true);
        ar.add(b.tpart[0], 2 * 3 * nmt * Bp * se, true);
        ar.add(b.tpart[1], 2 * 3 * nmt * Bp * se, true);
        ar.add(b.tDop, 2 * C2 * P * op, false);
        ar.add(b.ts[1], 2 * 3 * Bp * P * se, false);
        ar.add(b.tdlt, 2 * 3 * Bp * P * se, false);
        ar.add(b.tY, 2 * 2 * Bp * P * se, false);
    }
}

void add_decay_buffers(const Geometry& g, EnsembleBuffers& b, Arena& ar) {
    const size_t ge = (size_t)gemm_elt_bytes(g.precision), se = (size_t)state_elt_bytes(g.precision);
    const size_t P = (size_t)g.P, Bp = (size_t)g.Bp, op = ge * (size_t)operand_split(g.precision);
    ar.add(b.gmom, 18 * Bp * sizeof(double), true);
    ar.add(b.AG, P * P * op, false);
    ar.add(b.AGG, P * P * op, false);
    ar.add(b.Zop, Bp * P * op, false);
    ar.add(b.GX, 2 * Bp * P * se, false);
    ar.add(b.UZ, Bp * P * se, false);
    ar.add(b.dg, P * se, false);
}

Geometry make_geometry(int precision, int cfg, int64_t N, int64_t B) {
    Geometry g;
    g.precision = precision;
    g.cfg = cfg;
    const TileCfg& tc = tile_cfg(precision, cfg);
    g.kt = tc.kbytes / gemm_elt_bytes(precision);
    g.N = N;
    g.B = B;
    // whole tiles and ring stages
    g.P = round_up(N, std::max<int64_t>(tc.mt, g.kt * tc.group));
    g.Bp = round_up(B, tc.nt / 2);
    g.nmt = g.P / tc.mt;
    g.C2 = 2 * g.Bp;
    return g;
}

}  // namespace twa

// ===========================================================================
extern "C" {

TWA_API const char* twa_last_error(void) { return twa::g_err.c_str(); }
TWA_API const char* twa_version(void) { return "twa-mi355x 0.1 (gfx950)"; }

TWA_API void twa_params_default(twa_params* p) {
    if (!p) return;
    std::memset(p, 0, sizeof(*p));
    p->gamma = 1.0;
    p->s0z = 1.0;
    p->burnin = -1;
    p->integrator = TWA_INT_HEUN;
    p->precision = TWA_PREC_FP32;
    p->n_lags = 0;
    p->lag_stride = 0;
    p->point = 0;
    p->tile_config = -1;
    p->stream = nullptr;
    p->init_state = nullptr;
    p->timing = 0;
    p->use_graph = 1;
    p->kappa = 0.25;
    p->adjoint_objectives = 0;
    p->pump_path = TWA_PUMP_DENSE;
    p->norm_tol = 1e-2;
}

TWA_API int twa_philox(const uint32_t* ctr, int64_t n, uint32_t key0, uint32_t key1, uint32_t* out, void* stream) {
    TWA_API_LOCK();
    if (n < 0 || (n > 0 && (!ctr || !out))) {
        twa::set_error("twa_philox: bad arguments");
        return TWA_EINVAL;
    }
    int rc = twa::launch_philox(ctr, n, key0, key1, out, (hipStream_t)stream);
    if (rc) return rc;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) {
        twa::set_error("twa_philox: kernel failed");
        return TWA_EHIP;
    }
    return TWA_OK;
}

TWA_API int twa_noise(uint64_t seed, int64_t step, int32_t point, int64_t n_traj, int64_t N, int32_t fp64,
                      double* zeta, double* g, void* stream) {
    TWA_API_LOCK();
    if (n_traj < 1 || N < 1 || step < 0 || !zeta || !g) {
        twa::set_error("twa_noise: bad arguments");
        return TWA_EINVAL;
    }
    int rc = twa::launch_noise_debug(seed, step, point, n_traj, N, fp64, zeta, g, (hipStream_t)stream);
    if (rc) return rc;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) {
        twa::set_error("twa_noise: kernel failed");
        return TWA_EHIP;
    }
    return TWA_OK;
}

TWA_API int twa_run(const twa_params* p, int64_t n_traj, double dt, int64_t n_steps, uint64_t seed,
                    twa_observables* out, const twa_outputs* outs) {
    TWA_API_LOCK();
    return twa::run_single(p, n_traj, dt, n_steps, seed, out, outs);
}

}  // extern "C"
