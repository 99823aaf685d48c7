// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/twa.h"

namespace twa {

// ---------------------------------------------------------------------------
// error plumbing
void set_error(const std::string& msg);

// Every entry point that touches the device holds this process-wide lock for
// its whole duration (recursive: the threshold search and the batch call
// other entry points).  hipFree synchronises the whole device, and a
// device-wide synchronisation while another thread's stream is being
// captured into a graph breaks that capture; serialising the calls keeps
// every free, allocation and pump build of one call out of another call's
// graph capture.
std::recursive_mutex& api_mutex();
#define TWA_API_LOCK() std::lock_guard<std::recursive_mutex> twa_api_lock_(::twa::api_mutex())
struct Status {
    int code = TWA_OK;
    std::string msg;
};
#define TWA_HIP_CHECK(expr)                                                       \
    do {                                                                          \
        hipError_t _e = (expr);                                                   \
        if (_e != hipSuccess) {                                                   \
            ::twa::set_error(std::string(#expr) + ": " + hipGetErrorString(_e));  \
            return TWA_EHIP;                                                      \
        }                                                                         \
    } while (0)

// ---------------------------------------------------------------------------
// tile configurations of the channel-mixing contraction.  A configuration is
// (MT rows of spins, NT operand columns = NT/2 trajectories x 2 components,
// K bytes per LDS stage, waves along M, waves along N, LDS stages, ...).
// A ring stage holds `group` K stages of one sweep.  With split > 1 as many
// groups of waves share them.  The order in which the spins of a trajectory
// are summed follows from mt, waves_m and `sums` (thread groups that add the
// tiles' partial sums), and nothing else of a configuration shows in a result.
// Configurations 0 to 8 (FP64: 0 to 3) are those a caller may ask for and keep
// their shapes (saved tune files name them).  9 and 10 are taken by the
// automatic choice only: narrower tiles with the row shape of 1 and 2, and so
// with their results bit for bit (FP64: 32x32, and 64x64 with two groups of
// waves).  A run reports them as `base`.
struct TileCfg {
    int mt, nt, kbytes, waves_m, waves_n, nstage, group, split, sums, base;
};
constexpr int kTileCfgs = 11, kPublicTileCfgs = 9;
constexpr TileCfg kTiles[4][kTileCfgs] = {
    // The 64x64 ring of three stages lets three blocks share a compute unit
    // (BF16 us a step with three and four stages: 201 x 500 14.1 and 13.7, 700 x
    // 512 21.6 and 20.7, 200 x 20000 103 and 118, 760 x 8000 204 and 219; FP32 200
    // x 20000 194 and 206; split BF16 167 and 184).
    // BF16, FP16
    {{16, 32, 64, 1, 1, 8, 1, 1, 4, 0}, {64, 64, 64, 2, 2, 3, 2, 1, 8, 1}, {128, 128, 128, 2, 2, 4, 1, 1, 4, 2},
     {128, 128, 64, 2, 2, 8, 1, 1, 4, 3}, {256, 128, 64, 4, 1, 6, 1, 1, 4, 4}, {128, 256, 64, 2, 2, 6, 1, 1, 2, 5},
     {256, 128, 64, 4, 2, 4, 1, 1, 8, 6}, {320, 256, 128, 4, 2, 2, 1, 1, 4, 7}, {320, 256, 64, 4, 2, 4, 1, 1, 4, 8},
     {64, 32, 64, 2, 1, 4, 2, 1, 8, 1}, {128, 64, 64, 2, 2, 4, 1, 1, 4, 2}},
    // split BF16
    {{16, 32, 64, 1, 1, 8, 1, 1, 4, 0}, {64, 64, 64, 2, 2, 3, 2, 1, 8, 1}, {128, 128, 64, 2, 4, 8, 1, 1, 4, 2},
     {128, 128, 64, 2, 2, 8, 1, 1, 4, 3}, {256, 128, 64, 4, 1, 6, 1, 1, 4, 4}, {128, 256, 64, 2, 2, 6, 1, 1, 2, 5},
     {256, 128, 64, 4, 2, 4, 1, 1, 8, 6}, {320, 256, 128, 4, 2, 2, 1, 1, 4, 7}, {320, 256, 64, 4, 2, 4, 1, 1, 4, 8},
     {64, 32, 64, 2, 1, 4, 2, 1, 8, 1}, {128, 64, 64, 2, 2, 4, 1, 1, 4, 2}},
    // FP32
    {{16, 32, 64, 1, 1, 8, 1, 1, 4, 0}, {64, 64, 64, 2, 2, 3, 2, 1, 8, 1}, {128, 128, 64, 2, 4, 8, 1, 1, 4, 2},
     {128, 128, 64, 2, 2, 8, 1, 1, 4, 3}, {256, 128, 64, 4, 1, 6, 1, 1, 4, 4}, {128, 256, 64, 2, 2, 6, 1, 1, 2, 5},
     {256, 128, 64, 4, 2, 4, 1, 1, 8, 6}, {320, 256, 128, 4, 2, 2, 1, 1, 4, 7}, {320, 256, 64, 4, 2, 4, 1, 1, 4, 8},
     {64, 32, 64, 2, 1, 4, 2, 1, 8, 1}, {128, 64, 64, 2, 2, 4, 1, 1, 4, 2}},
    // FP64 (configurations 0 to 3, 9 and 10 only).  The smallest tiles' rings
    // are as deep as lets four and three blocks share a compute unit, no more:
    // with five a unit at times got more than its share while others idled
    // (16x32, stage 1 at 600 x 400 50 us in place of 40).
    {{16, 32, 64, 1, 1, 10, 1, 1, 4, 0}, {64, 64, 64, 2, 2, 4, 2, 1, 8, 1}, {128, 128, 128, 2, 2, 4, 1, 1, 4, 2},
     {128, 128, 64, 2, 2, 8, 1, 1, 4, 3}, {}, {}, {}, {}, {},
     {32, 32, 64, 2, 1, 11, 1, 1, 8, 0}, {64, 64, 64, 2, 2, 4, 4, 2, 16, 1}},
};
// row of kTiles of a precision
constexpr int tile_table(int precision) {
    return precision == TWA_PREC_FP64 ? 3 : precision == TWA_PREC_FP32 ? 2 : precision == TWA_PREC_BF16X3 ? 1 : 0;
}
// Whether the corrector's launch may carry the next step's noise.  A noise
// block takes the LDS of a tile: where only one fits on a compute unit (256x128
// and 320x256) their short lives follow one another there, and a launch of
// their own is shorter (4096 x 1024 on 256x128 tiles: 100 us more of stage 2
// with them, 17 for the launch).
constexpr bool noise_fits(int mt, int nt, int kbytes, int nstage, int group) {
    return nstage * group * (mt + nt) * kbytes <= 80 * 1024 || mt * nt <= 64 * 64;
}
// whether a caller may ask for a configuration
inline bool tile_cfg_ok(int precision, int id) { return id < (precision == TWA_PREC_FP64 ? 4 : kPublicTileCfgs); }
const TileCfg& tile_cfg(int precision, int id);
int pick_tile_cfg(int precision, int64_t N, int64_t n_traj);

inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }
int gemm_elt_bytes(int precision);
int state_elt_bytes(int precision);
int operand_split(int precision);   // bf16 parts per operand value (split BF16 2, else 1)

// ---------------------------------------------------------------------------
// device buffers and launch geometry of one trajectory ensemble
struct Geometry {
    int precision;
    int cfg;
    int integrator = TWA_INT_HEUN;
    int coh = 0;         // coherent exchange: operand columns (s | zeta | s_perp), corrector [D | D_perp]
    int64_t N, B;        // atoms, trajectories
    int64_t P, Bp;       // padded
    int64_t nmt;         // P / MT
    int64_t C2;          // 2 * Bp operand columns
    int64_t kt;          // K elements per LDS stage
};

// Device buffers of one call, carved from one allocation: the pieces that
// have to start at zero lie first and are cleared by one memset.  One
// hipMalloc, memset and hipFree instead of twenty each (a call of 64 steps at
// N = 10 took 480 us, most of it these).
class Arena {
  public:
    Arena() = default;
    Arena(const Arena&) = delete;
    Arena& operator=(const Arena&) = delete;
    ~Arena() { release(); }
    template <typename T>
    void add(T*& p, size_t bytes, bool zero) {
        items_.push_back({reinterpret_cast<void**>(&p), bytes, zero});
    }
    // allocates, sets the pointers and clears on st.  keep: the block may be
    // the one kept from an earlier call and is kept after this one (only for
    // calls that wait for their stream before they release).
    int commit(bool keep, hipStream_t st);
    void release();
    // the block without its owner, whose caller frees it
    void* detach();

  private:
    struct Item {
        void** p;
        size_t bytes;
        bool zero;
    };
    std::vector<Item> items_;
    void* block_ = nullptr;
    size_t bytes_ = 0;
    bool keep_ = false;
};
// hipMalloc that gives back the kept block and tries again if memory is short
hipError_t device_malloc(void** p, size_t bytes);
template <typename T>
hipError_t device_malloc(T** p, size_t bytes) {
    return device_malloc(reinterpret_cast<void**>(p), bytes);
}
// The kept block lives as long as any pump handle does, holds at most a 64th
// of the device's memory and is only touched under the API lock.  A call that
// needs less than an eighth of a large one gives it back and keeps its own.
void kept_block_free();
size_t kept_block_bytes();
void pump_born();
void pump_gone();

struct EnsembleBuffers {
    void* block = nullptr;      // the allocation of a batch point's buffers (single runs: the call's Arena)
    void* A = nullptr;          // GT [P][2P]  = [-dt/2 W | -sqrt(dt) F]
                                //    coherent exchange: [P][3P] = [-dt/2 W | -sqrt(dt) F | dt Omega]
    void* A2 = nullptr;         // GT [P][2P]  coherent exchange only: [-dt/2 W | dt Omega] (corrector)
    void* Xop = nullptr;        // GT [C2][2P] rows: (s^a | zeta^a) of one column; coherent exchange
                                //    [C2][3P] with s_perp = (s^y, -s^x) for the (x, y) columns
    void* Dop = nullptr;        // GT [C2][P]  predictor increments (coherent exchange [C2][2P]: D, D_perp)
    void* s[2] = {nullptr, nullptr};   // ST [3][Bp][P] ping-pong state
    void* dlt = nullptr;        // ST [3][Bp][P] predictor increment (kept only where response copies need it)
    void* Sn = nullptr;         // ST [2][Bp] collective sums S^x, S^y of the step's input state
    void* Y = nullptr;          // ST [2][Bp][P] contraction output of stage 1 (and 2)
    void* part[2] = {nullptr, nullptr};// ST [3][nmt][Bp] partial spin sums: [0] current state, [1] predictor
    void* g = nullptr;          // ST [2][2][Bp] collective normals of the steps of either parity
    bool ahead = false;         // stage 2 makes the next step's noise (into the other parity's normals),
                                // stage 1 observes the state it starts from where fold is set
    bool fold = false;
    void* norm0 = nullptr;      // ST [Bp][P]
    void* mom = nullptr;        // ST [5][2][Bp] Kahan (sum, compensation)
    // response copies (two-time)
    void* tXop = nullptr;       // GT [2][C2][P]
    void* tDop = nullptr;       // GT [2][C2][P]
    void* ts[2] = {nullptr, nullptr};  // ST [2][3][Bp][P]
    void* tdlt = nullptr;       // ST [2][3][Bp][P]
    void* tY = nullptr;         // ST [2][2][Bp][P]
    void* tpart[2] = {nullptr, nullptr};// ST [2][3][nmt][Bp]
    void* sm0 = nullptr;        // ST [2][Bp]
    double* lag = nullptr;      // [L][J][6]
    // correlated decay (model handles)
    void* AG = nullptr;         // GT [P][P] G
    void* AGG = nullptr;        // GT [P][P] G o G (elementwise square)
    void* Zop = nullptr;        // GT [Bp][P] packed s^z operand
    void* GX = nullptr;         // ST [2][Bp][P] G s^x, G s^y
    void* UZ = nullptr;         // ST [Bp][P] (G o G) s^z
    void* dg = nullptr;         // ST [P] diagonal of G
    double* gmom = nullptr;     // [9][2][Bp] Kahan (sum, compensation) of the estimator quantities
    int64_t* step = nullptr;    // device step counter; [1]: the next step, written by stage 1 (ahead)
    float* diag = nullptr;      // per-block max norm deviation / nan flags
};

struct StepConsts {
    double c1;      // Gamma dt / 2
    double c2;      // sqrt(Gamma dt)
    double s0z;
    uint32_t key0, key1;
    int32_t point;
    int64_t burnin, lag_stride, n_lags;
    int J;
};

// Type-erased description of one contraction launch (pointers are device
// buffers of the geometry's precision; kinds: 0 primal, 1 response tangent,
// 2 store (out = in + sign * A X), 3 adjoint of the corrector, 4 adjoint of
// the predictor, 5 semi-implicit, KIND_PRIMAL_WITH_Q the predictor that also
// stores the contribution of the second K half into Sout).
constexpr int KIND_PRIMAL_WITH_Q = 0x100;
struct GemmCall {
    int kind = 0, stage = 1, ncopy = 1;
    const void* A = nullptr;        // P rows, stage-blocked (a_index, the geometry's kt)
    const void* X = nullptr;        // columns, stage-blocked (x_index)
    int64_t x_copy = 0, K = 0;      // K: operand elements of one row along the contraction (all parts)
    double c1 = 0, c2 = 0;
    const void* s_cur = nullptr;
    void *s_next = nullptr, *dlt = nullptr, *Y = nullptr, *Y2out = nullptr, *Dop = nullptr, *Xnext = nullptr;
    const void* part_prim = nullptr;
    void* part_out = nullptr;
    const void* g = nullptr;
    int store_y2 = 0;
    const void* tpart_in = nullptr;
    int64_t* step = nullptr;
    const void* Sin = nullptr;
    void* Sout = nullptr;
    double store_sign = 1.0;
    const void *Y2in = nullptr, *Qin = nullptr, *YA = nullptr;
    void *lam = nullptr, *M1 = nullptr, *Rb = nullptr;
    double* gacc = nullptr;
    double inv_w = 0;
    // response / parameter tangent copies (kind 1): their state, increment,
    // field and operands; with Qin set, kind 1 adds the w-source Y/w - Q/(2w)
    const void* t_cur = nullptr;
    void *t_next = nullptr, *t_dlt = nullptr, *tY = nullptr, *tDop = nullptr;
    double srccoef[2][5] = {{0}};
    double src_scale = 0;
    int src_on = 0;
};
int launch_gemm_call(const Geometry& g, const GemmCall& c, hipStream_t st);

// Grouped persistent contraction launches over many ensembles that share a
// precision and tile configuration (one launch per stage covers all of them).
// Variants of a stage: the plain primal step, the primal step inside a
// two-time window (predictor increment kept, corrector field stored for the
// response copies) and the two response copies themselves.
enum { GV_PRIMAL = 0, GV_PRIMAL_TAN = 1, GV_TANGENT = 2, GV_COUNT = 3 };
struct GroupedPlan {
    void* d_args[GV_COUNT][2][2] = {};   // [variant][stage-1][cur] per-ensemble arguments
    // (point, M tile, column tile, copy): [0] stage 1, with observation blocks
    // (point, block, -, -1); [1] both response copies; [2] stage 2, with noise blocks
    int4* d_tiles[3] = {nullptr, nullptr, nullptr};
    int ntiles[3] = {0, 0, 0};
    int grid[3] = {0, 0, 0};
    int cfg = 0, precision = 0, integrator = TWA_INT_HEUN;
    bool tangents = false;
    int64_t* step = nullptr;
};
int grouped_prepare(const std::vector<Geometry>& gs, const std::vector<EnsembleBuffers>& bs,
                    const std::vector<StepConsts>& cs, int64_t* step, bool tangents, GroupedPlan& pl,
                    hipStream_t st);
// per-precision launchers, instantiated one precision per translation unit
// (twa_step_<precision>.hip); launch_gemm, launch_gemm_call, grouped_prepare
// and grouped_launch dispatch to them
template <int PREC>
int launch_gemm_p(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, int stage, bool tangent, int cur,
                  bool store_y2, bool keep_dlt, hipStream_t st);
template <int PREC>
int launch_call_p(const Geometry& g, const GemmCall& c, hipStream_t st);
template <int PREC>
int grouped_prepare_p(const std::vector<Geometry>& gs, const std::vector<EnsembleBuffers>& bs,
                      const std::vector<StepConsts>& cs, int64_t* step, bool tangents, GroupedPlan& pl,
                      hipStream_t st);
template <int PREC>
int grouped_launch_p(const GroupedPlan& pl, int stage, int cur, int variant, hipStream_t st);
int grouped_launch(const GroupedPlan& pl, int stage, int cur, int variant, hipStream_t st);
void grouped_free(GroupedPlan& pl);

// kernel launchers (twa_step.hip, twa_aux.hip)
int launch_build_A(const Geometry& g, const double* W, const double* F, double dt, void* A, hipStream_t st);
int launch_build_A_coh(const Geometry& g, const double* W, const double* F, const double* Om, double dt, void* A,
                       void* A2, hipStream_t st);
// (Xop null: a path that contracts nothing)
int launch_init_state(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c,
                      const double* init_dev, hipStream_t st);
int launch_reduce_state(const Geometry& g, const void* s, void* part, hipStream_t st);
inline bool noise_ahead(const Geometry& g) {
    const TileCfg& t = tile_cfg(g.precision, g.cfg);
    return noise_fits(t.mt, t.nt, t.kbytes, t.nstage, t.group);
}
int launch_noise(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, hipStream_t st);
int launch_gemm(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, int stage,
                bool tangent, int cur, bool store_y2, bool keep_dlt, hipStream_t st);
int launch_seed_tangents(const Geometry& g, const EnsembleBuffers& b, int cur, hipStream_t st);
int launch_observe(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, int cur,
                   bool tangents, hipStream_t st);
int launch_finish(const Geometry& g, const EnsembleBuffers& b, int cur, int nblk, hipStream_t st);
int launch_export_state(const Geometry& g, const void* s, double* out_dev, hipStream_t st);
int launch_advance_step(int64_t* step, hipStream_t st);
int launch_philox(const uint32_t* ctr, int64_t n, uint32_t k0, uint32_t k1, uint32_t* out, hipStream_t st);
int launch_noise_debug(uint64_t seed, int64_t step, int32_t point, int64_t B, int64_t N, int fp64,
                       double* zeta, double* g, hipStream_t st);

// fused small-N path (twa_small.hip): every step in one launch
bool small_path_applies(int precision, int64_t N, int64_t n_lags);
int launch_small_run(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, const twa_pump* pump,
                     double dt, int64_t n_steps, int out_cur, hipStream_t st);

// correlated decay (twa_decay.hip): observation operands and the per-step
// estimator of correlated emission; the geometry pads trajectories to a
// multiple of the column tile
int decay_geometry_ok(const Geometry& g);
int launch_decay_ops(const Geometry& g, const double* G, const EnsembleBuffers& b, hipStream_t st);
int launch_decay_observe(const Geometry& g, const EnsembleBuffers& b, int cur, hipStream_t st);

// Toeplitz fast path (twa_toeplitz.hip): circulant embedding of Eq. (2), one
// workgroup per trajectory over chunks of steps
int toeplitz_embedding_log2(int64_t N);
double toeplitz_spectrum_max(int64_t N, double w, double alpha);
int64_t toeplitz_max_n(int precision);
size_t toeplitz_table_bytes(const Geometry& g);
int toeplitz_tables(const Geometry& g, double w, double alpha, double dt, void* tw, void** spec, hipStream_t st);
int launch_toeplitz_run(const Geometry& g, const EnsembleBuffers& b, const StepConsts& c, const void* tw,
                        const void* spec, int64_t n_steps, int cur, hipStream_t st);

// pump (twa_pump.hip): the Eq. (2) pump of a handle rescaled to amplitude w
int pump_scaled(const twa_pump* base, double w, twa_pump** out);
// sum over the nmt M-tile partials of trajectory k in tile order, for the
// channels c0 .. c0 + NC - 1; the loads of eight tiles are issued before
// their additions (the order of the additions is unchanged)
template <typename S, int NC>
__device__ __forceinline__ void tile_sums(const S* part, int64_t nmt, int64_t Bp, int64_t k, int c0, S (&out)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) out[c] = 0;
    int64_t q = 0;
    for (; q + 8 <= nmt; q += 8) {
        S v[NC][8];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < 8; ++u) v[c][u] = part[((c0 + c) * nmt + q + u) * Bp + k];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < 8; ++u) out[c] += v[c][u];
    }
    for (; q < nmt; ++q)
#pragma unroll
        for (int c = 0; c < NC; ++c) out[c] += part[((c0 + c) * nmt + q) * Bp + k];
}

// v added to a Kahan-compensated sum
template <typename S>
__device__ __forceinline__ void kahan_add(S* sum, S* comp, S v) {
    const S s = *sum, c = *comp;
    const S y = v - c;
    const S t = s + y;
    *comp = (t - s) - y;
    *sum = t;
}

// the window moments (T2, T3, T4, Z, ZZ) of one trajectory's spin sums added to
// its time sums mom [5][2][Bp]
template <typename S>
__device__ __forceinline__ void add_moments(const S (&s)[3], S* mom, int64_t Bp, int64_t k) {
    const S T2 = S(0.25) * (s[0] * s[0] + s[1] * s[1]);
    const S v[5] = {T2, T2 * s[2], T2 * T2, s[2], s[2] * s[2]};
#pragma unroll
    for (int m = 0; m < 5; ++m) kahan_add(mom + (2 * m) * Bp + k, mom + (2 * m + 1) * Bp + k, v[m]);
}

}  // namespace twa

struct twa_pump {
    int64_t N;
    double w, alpha;
    double lam_min, lam_max;
    double* W = nullptr;     // device FP64 [N][N]
    double* F = nullptr;     // device FP64 [N][N]
    double* V = nullptr;     // device FP64 eigenvectors, column-major (column j = vector j)
    double* lam = nullptr;   // host eigenvalues ascending [N]
    double* G = nullptr;     // device FP64 [N][N] correlated-decay matrix (model handles only); then
                             // W holds the drift matrix W - G and F, V, lam belong to W + G
    double* Om = nullptr;    // device FP64 [N][N] coherent exchange Omega (model handles, optional)
    int device = 0;
    twa_pump() { twa::pump_born(); }
    twa_pump(const twa_pump&) = delete;
    ~twa_pump() { twa::pump_gone(); }
};
