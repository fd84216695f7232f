// Internal declarations shared by the translation units of liboco (host API,
// dense-round kernel, sparse-round kernel, meta/finalize kernels).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

namespace oco {

constexpr int kWave = 64;          // gfx950 wavefront width
constexpr float kFoldLo = 0x1p-24f; // lazy scale is folded into the vector outside [lo, hi]
constexpr float kFoldHi = 0x1p+24f;

// Z holds, for the rounds of one oco_run_rounds call, the prediction
// z_t^i = <w_t^i, x_t> of every base learner (i < K) and of the comparator
// (i == K).  Element (r, i, t) lives at Z[r*zs_r + i*zs_i + t*zs_t].
struct ZLayout {
    int64_t zs_r, zs_i, zs_t;
};

// Tuning choices of a state (oco_set_option), indexed by oco_option; -1 = the library decides.
constexpr int kNumOptions = 12;
struct Tuning {
    int64_t v[kNumOptions];
    __host__ Tuning() { for (auto &e : v) e = -1; }
    int64_t get(int key) const { return v[key]; }
};

// How the dense round kernel of a state is launched: depends on the configuration and the
// tuning choices only (not on n or t0), so it is worked out once and kept in the state.
struct DensePlanCache {
    bool valid = false;
    const void *kern = nullptr;
    size_t smem = 0;
    int wpb = 0, rt = 0, rt0 = 0;
    int64_t nwg = 0, batches = 0;
    int per_run = 0;
    bool after_split = false;    // the call before was worked by dense_split.hip or dense_run.hip (not part of the plan: survives a change of options)
};

// Called after the round kernel of every piece of a call has been enqueued: rounds
// [off, off + len) of the call have their predictions in Z once that kernel finishes.
struct PieceHook {
    hipError_t (*fn)(void *ctx, int off, int len);
    void *ctx;
    // Optional: a stream for work of the call that the round kernels neither wait for nor feed
    // (it starts after the work already on the call's stream, and what fn enqueues follows it).
    hipError_t (*beside)(void *ctx, hipStream_t *out) = nullptr;
    // Optional, with `beside`: mark remembers what is on that stream now; after wait_mark the call's stream
    // goes on only when that work is done (for work beside the round kernels that a later one of them needs).
    hipError_t (*mark)(void *ctx) = nullptr;
    hipError_t (*wait_mark)(void *ctx) = nullptr;
};

// Event pairs around the launches of a call's dominant kernel (benchmarks: the duration of that
// kernel alone, launch by launch).  The launchers call begin / end around each such launch; with
// no clock, or past its capacity, they cost nothing and only count.
struct LaunchClock {
    static constexpr int kPairs = 64;
    hipEvent_t ev[2 * kPairs] = {};
    int launches = 0;          // of the last call
    int timed = 0;             // of those, how many have an event pair
    const char *kernel = "";   // which kernel the launcher timed
    hipError_t begin(hipStream_t s) { return timed < kPairs && ev[2 * timed] ? hipEventRecord(ev[2 * timed], s) : hipSuccess; }
    hipError_t end(hipStream_t s)
    {
        ++launches;
        if (timed >= kPairs || !ev[2 * timed + 1]) return hipSuccess;
        return hipEventRecord(ev[2 * timed++ + 1], s);
    }
};
inline hipError_t clock_begin(LaunchClock *c, hipStream_t s, const char *kernel)
{
    if (!c) return hipSuccess;
    c->kernel = kernel;
    return c->begin(s);
}
inline hipError_t clock_end(LaunchClock *c, hipStream_t s) { return c ? c->end(s) : hipSuccess; }

// ---- dense rounds -----------------------------------------------------------
struct DenseArgs {
    const float *x;          // round stream (or gradient stream for the linear loss)
    int64_t x_run_stride;    // elements between runs (unused when x_shared)
    const float *y;          // labels, may be null (linear loss)
    int64_t y_run_stride;
    const float *u;          // comparator segments [R][S][d]
    const int64_t *seg_start;// device copy, [S]
    int S;
    float *V;                // [R][K][d]  iterate = sigma * V
    float *sigma;            // [R][K]
    double *n2;              // [R][K]  ||V row||^2
    float *x2;               // scratch: ||x_t||^2 per round of this call, [n] or [R][x2_run_stride]
    int64_t x2_run_stride;
    const float *eta;        // [K]
    float *Z;
    ZLayout zl;
    int d, K, R;
    int64_t t0;              // absolute index of the first round of this call
    int n;                   // rounds in this call
    float D;
    int x_shared;
    int vec_ok;              // rows of x are 16-byte aligned and d % 4 == 0
    int per_run;             // wavefront tasks per run: K + 1 with the comparator's, K when its
                             // predictions come from the contraction kernel (set by the launcher)
    int rt;                  // rounds per tile of the register kernel's ring (set by the launcher)
    // A short call whose runs have a workgroup each is one kernel (dense_short.hip): its workgroups also take the norms
    // of the rounds (x2, g01), keep the last row and do the meta kernel's work on their run.
    double *L, *last, *regret;   // of the meta learner, as in MetaArgs
    double eps;
    // optimistic two-step update (Eq. (3)); V then holds the intermediate model w^
    int optimistic;
    float *ha;               // [R][K]  eta_i c_{t-1}^i: the hint is ha * x_{t-1}
    float *hp;               // [R][K]  <w^_t, x_{t-1}>
    float *g01;              // scratch like x2: <x_{t-1}, x_t> per round of this call
    float *xlast;            // [1 or R][d]  last round row of the previous call (0 before round 0)
    float *x2last;           // [1 or R]     its squared norm
    const Tuning *tune;      // never null
    LaunchClock *clock;      // null unless the call is timed
    DensePlanCache *plan;    // never null
    float *gram;             // shared streams: dense_gram_bytes(n_max, d) of scratch for the windowed path
    int64_t n_max;           // the state's largest call (lays that scratch out)
    int64_t T;               // the horizon
    bool scaled;             // chain_holds of the configuration
};

// Whether the dependent rounds in scaled coordinates (chain_rounds, dense_chain.h) hold a configuration of radius D whose steps
// are at most `step` long (the largest eta times the bound G of Assumption 2; the kernels that have them are not wanted otherwise).
//  - Squared norms are kept in float32 between windows, so D^2 has to be a normal float32.  (The other kernels never project where
//    it is infinite, as with a radius that stands for no bound at all; here the scale of the iterates, D / sqrt 2, would be infinite too.)
//  - The scale grows by 1 + r, r = step / D, in every round that leaves the ball and is taken back below 2 every eighth round if it is
//    beyond 2^20, so a squared norm reaches 2^40 D^2 (1 + r)^16, which has to stay within float64's 2^1024: 8 log2 r + log2 D < 491.
//    15 of these are left for gradients beyond G (3.6 times).  The step grid of Corollary 3 is within it at K = 64 for D <= 1000 (T >= 768).
inline bool chain_holds(double D, double step)
{
    if (!(D >= 0x1p-63 && D < 0x1p64)) return false;
    const double r = step / D;
    return r <= 1.0 || 8.0 * std::log2(r) + std::log2(D) < 476.0;
}
// *meta_done: the call's meta work is enqueued as well (a.L, a.last, a.regret)
hipError_t launch_dense_rounds(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook, bool *meta_done);
bool dense_short_supported(const DenseArgs &a);
hipError_t launch_dense_short(const DenseArgs &a, int loss, hipStream_t s);
// the windowed path (dense_window.hip): whether a configuration takes it, and its launcher
bool dense_window_wanted(const DenseArgs &a);
hipError_t launch_dense_window(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook);
// the windowed path with a tile's coordinates split over workgroups (dense_split.hip)
bool dense_split_wanted(const DenseArgs &a);
hipError_t launch_dense_split(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook);
// windows of a stream per tile of learners (dense_run.hip)
bool dense_run_wanted(const DenseArgs &a);
hipError_t launch_dense_run(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook);
hipError_t launch_hint_scalars(const DenseArgs &a, hipStream_t s);
hipError_t launch_keep_last_row(const DenseArgs &a, hipStream_t s);
size_t dense_gram_bytes(int64_t n_max, int64_t d);

// comparator predictions of a shared dense stream as one contraction (rows K of Z)
struct ComparatorGemmArgs {
    const float *x;          // [n][d]
    const float *u;          // [R][S][d]
    const int64_t *seg_start;// device, [S]
    int S;
    float *Z;
    ZLayout zl;
    int d, K, R;
    int64_t t0;
    int n;
    int vec_ok;              // rows of x and u are 16-byte aligned and d % 4 == 0
    int chunks = 1;          // ranges of coordinates summed apart, with
    float *part = nullptr;   // chunks R n floats of scratch (null: one range)
    bool fine = false;       // short float32 sums, added in float64 (vec_ok only)
};
hipError_t launch_comparator_gemm(const ComparatorGemmArgs &a, hipStream_t s);
bool dense_supported(int64_t d, int x_shared);

// ---- sparse rounds ----------------------------------------------------------
struct SparseArgs {
    const int32_t *col;      // [n][nnz]
    const float *val;        // [n][nnz]
    const float *y;
    int64_t y_run_stride;
    const float *u;          // [R][S][d]
    const int64_t *seg_start;
    int S;
    float *V;                // [d][RKp]: coordinate-major, the R*K learners interleaved (RKp: padded row length)
    double *sigma;           // [RKp]
    double *n2;              // [RKp]  ||V column||^2
    const float *eta;        // [K]
    float *Z;
    ZLayout zl;
    int d, K, R, nnz, RKp;
    int64_t t0;
    int n;
    double D;
    void *scratch;           // sparse_scratch_bytes(n_max) bytes: per-window Gram data of the call
    // optimistic two-step update (Eq. (3)); V then holds the intermediate model w^
    int optimistic;
    float *ha;               // [RKp]  eta_i c_{t-1}^i: the hint is ha * x_{t-1}
    float *hp;               // [RKp]  <w^_t, x_{t-1}>
    float *hx;               // [RKp]  ||x_{t-1}||^2 (the same for all learners; kept per lane)
    int32_t *last_col;       // [OCO_MAX_NNZ]  last round row of the previous call (zeros before round 0)
    float *last_val;         // [OCO_MAX_NNZ]
    float *xlast_dense;      // [d]  the same row scattered into a dense vector (for the export)
    const Tuning *tune;      // never null
    LaunchClock *clock;      // null unless the call is timed
};
hipError_t launch_sparse_rounds(const SparseArgs &a, int loss, hipStream_t s, const PieceHook *hook);
size_t sparse_scratch_bytes(int64_t n_max);

// ---- meta learner + regret --------------------------------------------------
struct MetaArgs {
    const float *Z;
    ZLayout zl;
    const float *y;
    int64_t y_run_stride;
    double *L;               // [R][K] cumulative losses, updated in place
    double *last;            // [R][K] last observed losses (the meta learner's hint), updated in place; or null
    double *regret;          // [R]
    double eps;
    int K, R, n;
};
hipError_t launch_meta(const MetaArgs &a, int loss, hipStream_t s);

// The losses (meta kernel and short dense calls).
template <int LOSS> __device__ __forceinline__ double phi(double z, double y)
{
    if (LOSS == 0) return z;
    if (LOSS == 1) { const double e = z - y; return e * e; }
    // log(1 + exp(-m)) without overflow: log1p(exp(-|m|)) + max(-m, 0).  One exp and one log1p
    // for every lane (a branch on the sign of m would run both sides in most wavefronts).
    const double m = y * z;
    const double am = fabs(m);
    const double lp = log1p(exp(-am));
    return m > 0.0 ? lp : lp + am;
}

// Their slopes, in float32 (round kernels).
template <int LOSS> __device__ __forceinline__ float slope(float z, float y)
{
    if (LOSS == 0) return 1.0f;
    if (LOSS == 1) return 2.0f * (z - y);
    // logistic: -y / (1 + exp(y z)); exp overflow gives -y * (1/inf) = -0
    return -y * __builtin_amdgcn_rcpf(1.0f + __expf(y * z));
}

// ---- state export -----------------------------------------------------------
struct ExportArgs {
    const float *V;
    const void *sigma;       // float [R][K] (dense) or double [RKp] (sparse)
    const double *L;
    const double *last;      // the meta learner's hint, or null
    double eps;
    float *W, *p, *wbar;     // any may be null
    int d, K, R, RKp;
    int sparse;
    // optimistic: the exported iterate is Proj[sigma V - ha xlast].  Dense: xlast [1 or R][d],
    // x2last [1 or R].  Sparse: xlast [d] (dense copy of the last sparse row), x2last [RKp].
    int optimistic;
    const float *ha, *hp, *xlast, *x2last;
    const double *n2;
    int x_shared;
    float D;
};
hipError_t launch_export(const ExportArgs &a, hipStream_t s);
hipError_t launch_accel_bounds(const double *regret, int R, int64_t t, int64_t k, double alpha, double *out,
                               hipStream_t s);

// step sizes as a kernel argument
struct EtaTable { float v[64]; };
hipError_t launch_set_eta(float *eta_dev, const EtaTable &tab, int K, hipStream_t s);

// fills `bytes` (a multiple of 16) of device memory with zero using a kernel,
// and sets every sigma to 1
hipError_t launch_init_state(void *zero_base, size_t zero_bytes, void *sigma, int64_t n_sigma,
                             int sigma_is_double, hipStream_t s);

}  // namespace oco
