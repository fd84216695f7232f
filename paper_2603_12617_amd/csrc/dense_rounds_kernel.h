// Dense rounds of the base learners (Sec. 3.1 update inside the ensemble of
// Sec. 3.3), many rounds per launch.
//
// Mapping.  One wavefront owns one base learner of one run for the whole call:
// lane l keeps d/64 coordinates of the iterate in registers, so the inner
// product <w_t^i, x_t> and the norm of the stepped vector are wavefront
// reductions (DPP) and no learner ever waits for another -- each base learner
// steps along the gradient at its own iterate.  One extra wavefront per run
// carries the comparator u_t and only takes inner products.  The wavefronts of
// a workgroup share the round stream: x is copied from global memory straight
// into an LDS ring of three tiles of RT rounds (global_load_lds, no staging
// registers), two tiles ahead of the compute, one barrier per tile.
//
// One pass over the registers per round.  The iterate is kept as w = sigma*v
// with a per-learner scalar sigma, so the projection onto the ball only
// changes sigma.  In round t the pass computes
//     v      <- v - b x_t,  b = eta c_t / sigma    (gradient step, c_t = phi'(z_t; y_t))
//     q      =  <v, x_{t+1}>                       (next round's prediction)
// and the norm needed by the projection follows from scalars already at hand,
//     ||v - b x_t||^2 = ||v||^2 - 2 b <v, x_t> + b^2 ||x_t||^2
// (<v, x_t> is the previous round's q, ||x_t||^2 comes from a small pre-pass
// over the round stream), carried in float32 like its inputs (float64 for the
// three scalars changed no result: the error is that of <v, x_t>) and
// re-measured exactly, as sum_j v_j^2 inside the pass, at every 64th round of
// the horizon so that rounding cannot accumulate.  Then sigma <- D/||v|| if sigma ||v|| > D, and
// z_{t+1} = sigma q.  x_{t+1} is
// read from LDS during the pass, one chunk ahead of the arithmetic, and stays
// in registers as the next round's x_t (two register sets that swap roles, the
// round loop is unrolled by two).  sigma is folded back into v, at the start of
// a round, once it has left [2^-24, 2^24].
//
// The kernel writes z_t^i for every round to Z; losses, Hedge weights and
// regret are computed from Z by the meta kernel.
#pragma once
#include "oco_internal.h"
#include "../../include/oco.h"

namespace oco {
namespace {

template <int NPL> struct DenseCfg;
// NPL: coordinates per lane.  MAXW: most wavefronts per workgroup (sets the register
// budget).  RT: rounds per LDS tile (even; RT*NPL a multiple of 4).
template <> struct DenseCfg<1>  { static constexpr int MAXW = 16, RT = 32; };
template <> struct DenseCfg<2>  { static constexpr int MAXW = 16, RT = 16; };
template <> struct DenseCfg<4>  { static constexpr int MAXW = 16, RT = 16; };
template <> struct DenseCfg<8>  { static constexpr int MAXW = 16, RT = 8; };
#ifndef OCO_RT16
#define OCO_RT16 2
#endif
template <> struct DenseCfg<16> { static constexpr int MAXW = 16, RT = OCO_RT16; };
#ifndef OCO_MAXW32
#define OCO_MAXW32 12
#endif
template <> struct DenseCfg<32> { static constexpr int MAXW = OCO_MAXW32, RT = 2; };
#ifndef OCO_MAXW64
#define OCO_MAXW64 12
#endif
template <> struct DenseCfg<64> { static constexpr int MAXW = OCO_MAXW64,  RT = 2; };
// One register set for the round row (x_t is replaced chunk by chunk with x_{t+1} as the step
// consumes it) instead of two that swap roles: 64 fewer registers per lane, which at 64
// coordinates per lane is the difference between two and three wavefronts per SIMD.
template <int NPL> constexpr bool kOneRowSet = NPL >= 64;   // at 32 it measured 4 % slower
constexpr int kRing = 3;   // LDS tiles
// Where the round loop of rows of at most 128 coordinates starts, in instructions of 4 bytes past a multiple of 64: a round
// there is so short that how its branch targets lie in the 32-byte blocks instructions are fetched in is up to 7 % of
// it, and left alone that changes with any code before the loop.  3000 plain rounds, us, best / worst of the sixteen
// offsets: two learners, d = 64, squared 593 / 638, logistic 662 / 704, linear 574 / 618 (13, 7, 15 / 3); eight runs of three on
// streams of their own, d = 96, 648 / 701, 721 / 768, 640 / 697 (6, 7, 6 / 1, 10, 12).
template <int NPL, int LOSS>
constexpr int kLoopOffset = NPL == 1 ? (LOSS == 1 ? 13 : 15) : NPL == 2 ? (LOSS == 2 ? 7 : 6) : -1;   // -1: wherever it falls
// Tiles may be longer than DenseCfg's.  Up to 128 coordinates theirs already outlast a load (4 us and more); longer
// ones cost 200 runs of 20 learners, d = 100, 5 % (1.41 -> 1.45 ms per 3000 rounds).
template <int NPL> constexpr bool kGrowTiles = NPL >= 4;

template <int VW> struct VecT;
template <> struct VecT<1> { using type = float; };
template <> struct VecT<2> { using type = float2; };
template <> struct VecT<4> { using type = float4; };

template <int VW> __device__ __forceinline__ void unpack(const typename VecT<VW>::type &t, float (&o)[VW])
{
    if constexpr (VW == 4) { o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w; }
    else if constexpr (VW == 2) { o[0] = t.x; o[1] = t.y; }
    else { o[0] = t; }
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_term(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

// Sum over the 64 lanes, result uniform.  Fixed order: xor-butterfly inside each row of
// 16 lanes, then rows 0+1 and 2+3, then the two halves.  The two cross-row steps are
// written as v_add_f32 with a DPP row broadcast and a row mask: rows outside the mask keep
// their value, so one instruction does what mov+mov_dpp+add would.  (A DPP operand needs
// two wait states after the VALU write that produced it, hence the s_nop.)
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_term<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_term<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    v += dpp_term<0x141, 0xF>(v);   // row_half_mirror
    v += dpp_term<0x140, 0xF>(v);   // row_mirror
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"   // rows 1, 3 += row 0, 2
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"   // rows 2, 3 += rows 0+1
        "s_nop 0"
        : "+v"(v));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Workgroup barrier that publishes the tiles copied global -> LDS.  Those copies complete
// asynchronously and are counted by vmcnt of the wavefront that issued them; a plain barrier
// does not wait for them (a workgroup-scope fence leaves vmcnt alone), and a wavefront that never
// reads the ring (padding wavefronts) would otherwise meet the barrier with its share of a tile
// still in flight.  Every wavefront therefore drains its own copies before it arrives.
__device__ __forceinline__ void tile_sync()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

template <int VW> __device__ __forceinline__ float combine(const float (&acc)[VW])
{
    if (VW == 4) return (acc[0] + acc[1]) + (acc[2] + acc[3]);
    if (VW == 2) return acc[0] + acc[1];
    return acc[0];
}

// Tile k of the ring for rows that are not 16-byte aligned (any d, any 4-byte address): copied straight to LDS
// like the aligned ones, a word per lane and 64 words of a row per instruction.  Four times the copy
// instructions of the aligned tiles, but asynchronous like those: read into registers and written to LDS,
// every tile waited for its own loads (d = 777, 240 learners: 1.6 us per round, now 0.8).  (A scalar row address
// with a lane offset, for these and the aligned copies: 5 % slower, the scalar index arithmetic is as long.)
template <int DP>
__device__ __forceinline__ void stage_words(const float *xg, int d, int n, int k, int RT, float *dst, int wave, int wpb, int lane)
{
    static_assert(DP % kWave == 0, "an instruction stays inside a row");
    for (int ii = wave; ii < RT * (DP / kWave); ii += wpb) {
        const int rr = ii / (DP / kWave), j = (ii % (DP / kWave)) * kWave + lane;
        const int tt = k * RT + rr;
        if (tt < n && j < d)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xg + (int64_t)tt * d + j),
                                             (__attribute__((address_space(3))) void *)(dst + ii * kWave), 4, 0, 0);
    }
}

// ||x||^2 of a round row and, if prev is given, its inner product with the row before: one wavefront, fixed order
// (one chain per sum).  The loads of U steps of 64 coordinates are issued together, U no larger than the row has
// steps left: a row of d = 64 taken as sixteen steps, fifteen of them empty, made the norms of 192000 rows 14.4 us
// instead of 8.4.  (Steps past the row add +0, which changes no bit of a sum of squares, and of the other at most the
// sign of a zero.)
template <int U, bool PREV, bool GUARD>
__device__ __forceinline__ void row_steps(const float *src, const float *prev, int j, int d, float &acc, float &ac2)
{
    float v[U], w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool in = !GUARD || j + 64 * u < d;
        v[u] = in ? src[j + 64 * u] : 0.f;
        if (PREV) w[u] = in ? prev[j + 64 * u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        acc = fmaf(v[u], v[u], acc);
        if (PREV) ac2 = fmaf(w[u], v[u], ac2);
    }
}
template <bool PREV>
__device__ __forceinline__ void row_sums(const float *src, const float *prev, int d, int lane, float &acc, float &ac2)
{
    int j = lane, left = d;                                // left: the same in every lane
    for (; left >= 64 * 16; left -= 64 * 16, j += 64 * 16) row_steps<16, PREV, false>(src, prev, j, d, acc, ac2);
    if (left > 64 * 4) row_steps<16, PREV, true>(src, prev, j, d, acc, ac2);
    else if (left > 64) row_steps<4, PREV, true>(src, prev, j, d, acc, ac2);
    else if (left > 0) row_steps<1, PREV, true>(src, prev, j, d, acc, ac2);
}
__device__ __forceinline__ void row_scalars(const float *src, const float *prev, int d, int lane, float &x2, float &g01)
{
    float acc = 0.f, ac2 = 0.f;
    if (prev) row_sums<true>(src, prev, d, lane, acc, ac2);
    else row_sums<false>(src, prev, d, lane, acc, ac2);
    x2 = wave_sum(acc);
    if (prev) g01 = wave_sum(ac2);
}

// ---- short calls -----------------------------------------------------------------------------
// A serving loop updates a learner after every few verification steps: calls of a handful of rounds, in which
// the launches around the rounds (norms, meta kernel on the second stream with its two waits, last row) are most
// of the time (one run of 3 learners, d = 1000, 8 rounds: 53 us per call of which the rounds are 8).  For at most
// kWholeRounds rounds, where a run's wavefronts fit one workgroup and the grid leaves the chip mostly idle, the
// workgroup of a run does that work itself; same arithmetic in the same order as the kernels it replaces (meta.hip),
// so the bits do not depend on how a horizon is cut.
constexpr int kWholeRounds = 64;

// LDS words behind the ring: ||x_t||^2, then <x_{t-1}, x_t>
constexpr int kWholeFloats = 2 * kWholeRounds;

// What wavefront 0 keeps for the meta work: the run's cumulative and last losses (a learner per lane) and its regret, loaded with
// everything else the kernel starts from.
struct WholeState { double L = 0.0, last = 0.0, regret = 0.0; };

// The meta kernel's work on run r for the n rounds of a short call: called by all wavefronts (wavefront i holds the
// predictions of learner i, i = K the comparator, a round per lane, and the labels; those behind only help) once the ring's space is free.
template <int LOSS>
__device__ __forceinline__ void whole_meta(const DenseArgs &a, float *ring, int r, int i, int lane, float zreg, float yreg, const WholeState &st)
{
    const int K = a.K, n = a.n;
    float *zs = ring;                                               // [K + 1][64]
    double *lm = reinterpret_cast<double *>(ring + (K + 1) * 64);   // [n][K]: losses, then cumulative losses before the round
    double *diff = lm + 64 * K;
    const double yt = (double)yreg;
    if (i <= K) zs[i * 64 + lane] = zreg;
    if (i < K && lane < n) lm[lane * K + i] = phi<LOSS>((double)zreg, yt);
    __syncthreads();
    const bool hint = a.last != nullptr;
    if (i == 0 && lane < K) {                                       // running sums in round order
        double Lacc = st.L, lprev = st.last;
        for (int t = 0; t < n; ++t) {
            const double l = lm[t * K + lane];
            lm[t * K + lane] = hint ? Lacc + lprev : Lacc;
            Lacc += l;
            lprev = l;
        }
        a.L[(int64_t)r * K + lane] = Lacc;
        if (hint) a.last[(int64_t)r * K + lane] = lprev;
    }
    __syncthreads();
    if (i == 0 && lane < n) {
        double Lmin = lm[lane * K];
        for (int k = 1; k < K; ++k) Lmin = fmin(Lmin, lm[lane * K + k]);
        double S = 0.0, zsum = 0.0;
        for (int k = 0; k < K; ++k) {
            const double e = exp(-a.eps * (lm[lane * K + k] - Lmin));
            S += e;
            zsum += e * (double)zs[k * 64 + lane];
        }
        diff[lane] = phi<LOSS>(zsum / S, yt) - phi<LOSS>((double)zs[K * 64 + lane], yt);
    }
    __syncthreads();
    if (i == 0 && lane == 0) {
        double reg = st.regret;
        for (int t = 0; t < n; ++t) reg += diff[t];
        a.regret[r] = reg;
    }
}

template <int NPL, int LOSS, bool OPT, bool WHOLE>
__global__ void __launch_bounds__(DenseCfg<NPL>::MAXW * kWave)
dense_rounds_kernel(const DenseArgs a)
{
    constexpr int VW = NPL >= 4 ? 4 : NPL;      // floats per LDS read
    constexpr int NV = NPL / VW;                // LDS reads per lane and round
    constexpr int DP = NPL * kWave;             // padded dimension
    // rounds per tile: even, divides 64; a constant where tiles never grow (tile_rounds)
    const int RT = kGrowTiles<NPL> ? a.rt : DenseCfg<NPL>::RT;
    const int TILE = RT * DP;                   // floats per tile
    const int NI = TILE / 4 / kWave;            // 1 KB copy instructions per tile
    constexpr int CH = NV >= 2 ? 2 : 1;         // LDS reads per chunk
#ifndef OCO_NACC64
#define OCO_NACC64 4
#endif
    // partial sums of the next-round dot: two chains (one add to combine them), four where the
    // chains would get 32 FMAs long
    constexpr int NACC = NPL >= 64 ? OCO_NACC64 : (VW >= 2 ? 2 : 1);
    constexpr int NCH = NV / CH;
    static_assert(DenseCfg<NPL>::RT * DP % (4 * kWave) == 0, "tile must be a whole number of 1 KB copies");
    static_assert(DenseCfg<NPL>::RT % 2 == 0, "the round loop is unrolled by two");
    using V = typename VecT<VW>::type;

    extern __shared__ float4 smem4[];
    float *ring = reinterpret_cast<float *>(smem4);

    const int tid = threadIdx.x;
    const int nthreads = blockDim.x;
    const int wpb = nthreads >> 6;              // wavefronts in this workgroup
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n;
    const int d = a.d;
    const int K = a.K;

    // ---- which task this wavefront owns: learner i < K, or the comparator (i == K) ----
    int r, i;
    bool active;
    if (WHOLE) {                              // a workgroup per run; wavefronts behind the run's tasks stage rows
        r = a.x_shared ? blockIdx.x : blockIdx.y;
        i = wave;
        active = i < a.per_run;
    } else if (a.x_shared) {
        const int64_t q = (int64_t)blockIdx.x * wpb + wave;
        active = q < (int64_t)a.R * a.per_run;
        r = active ? (int)(q / a.per_run) : 0;
        i = active ? (int)(q % a.per_run) : 0;
    } else {
        r = blockIdx.y;
        i = blockIdx.x * wpb + wave;
        active = i < a.per_run;
        if (!active) i = 0;
    }
    const bool is_cmp = active && i == K;
    const float *xg = a.x_shared ? a.x : a.x + (int64_t)blockIdx.y * a.x_run_stride;

    // ---- staging of x: tile k = rounds k*RT .. k*RT+RT-1 -> ring slot k % 3 ------
    auto issue_tile = [&](int k) {
        float *dst = ring + (k % kRing) * TILE;
        if (a.vec_ok) {
            for (int ii = wave; ii < NI; ii += wpb) {
                const int e = ii * kWave + lane;               // float4 index in the tile
                const int rr = e / (DP / 4), j4 = e % (DP / 4);
                const int tt = k * RT + rr;
                if (tt < n && j4 * 4 < d)
                    __builtin_amdgcn_global_load_lds(
                        (const __attribute__((address_space(1))) void *)(xg + (int64_t)tt * d + j4 * 4),
                        (__attribute__((address_space(3))) void *)(dst + ii * 4 * kWave), 16, 0, 0);
            }
        } else {
            stage_words<DP>(xg, d, n, k, RT, dst, wave, wpb, lane);
        }
    };

    // padding coordinates (j >= d) of the ring are never written again: zero them once (short calls: beside the loads, rows past the
    // call may hold anything, what is made of them is not used.  In long calls that saves nothing, and with it the instance for 8
    // coordinates per lane took 240 us for 614 rounds of 845 learners, 204 without)
    const int ntiles = (n + RT - 1) / RT;
    if (!WHOLE) {
        for (int e = tid; e < min(kRing, ntiles + 1) * TILE / 4; e += nthreads) smem4[e] = make_float4(0.f, 0.f, 0.f, 0.f);
        tile_sync();
    }
    issue_tile(0);
    if (ntiles > 1) issue_tile(1);
    if (WHOLE) {
        const int rows = min(kRing, ntiles + 1) * RT, rpi = nthreads >= DP ? nthreads / DP : 1;
        for (int row = tid / DP; row < rows && tid / DP < rpi; row += rpi)
            for (int j = d + tid % DP; j < DP; j += nthreads >= DP ? DP : nthreads) ring[row * DP + j] = 0.f;
    }
    float *whole_x2 = ring + kRing * TILE;
    // A short call is mostly latencies of loads, one behind the other: everything it starts from is on its way before the first barrier.
    // (With that, the last row kept beside the rounds and the ring cleared only where rows do not write it, a call of 8 optimistic rounds of 3
    // learners, d = 1000, is 11.1 us of this kernel, 13.3 before; 64 of them with the model read back after each 1084 -> 881 us.)
    // (The vector itself not beyond 2048 coordinates: there it would be spilled.)
    constexpr bool PRE = WHOLE && !kOneRowSet<NPL>;
    float first[PRE ? NV : 1][VW];              // V row of a learner, u of the comparator
    float sigma0 = 0.f, eta0 = 0.f, ha0 = 0.f, hp0 = 0.f, x2last0 = 0.f, y0 = 0.f;
    double n20 = 0.0;
    WholeState ws;
    int seg0 = 0;
    if (WHOLE && active) {
        const float *src;
        if (is_cmp) {
            while (seg0 + 1 < a.S && a.seg_start[seg0 + 1] <= a.t0) ++seg0;
            src = a.u + ((int64_t)r * a.S + seg0) * d;
        } else {
            const int64_t q = (int64_t)r * K + i;
            src = a.V + q * d;
            sigma0 = a.sigma[q];
            n20 = a.n2[q];
            eta0 = a.eta[i];
            if (OPT) { ha0 = a.ha[q]; hp0 = a.hp[q]; x2last0 = a.x2last[a.x_shared ? 0 : r]; }
            if (a.y && lane < n) y0 = a.y[(int64_t)r * a.y_run_stride + lane];
            if (i == 0) {
                if (lane < K) { ws.L = a.L[q + lane]; if (a.last) ws.last = a.last[q + lane]; }
                if (lane == 0) ws.regret = a.regret[r];
            }
        }
        if constexpr (PRE) {
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    const int j = (m * kWave + lane) * VW + e;
                    first[m][e] = j < d ? src[j] : 0.f;
                }
        }
    }
    if (WHOLE) {
        for (int t = wave; t < n; t += wpb) {
            const float *src = xg + (int64_t)t * d;
            float x2, g01 = 0.f;
            row_scalars(src, OPT ? (t > 0 ? src - d : a.xlast + (a.x_shared ? 0 : (int64_t)r * d)) : nullptr, d, lane, x2, g01);
            if (lane == 0) { whole_x2[t] = x2; whole_x2[kWholeRounds + t] = g01; }
        }
    }
    tile_sync();
    // The last row, for the next call's hint (the only workgroup that read the old one, before the barrier; the launcher does not send a
    // shared stream of several runs here): by the first wavefront without a task, beside the last tile's rounds, if there is one.
    auto keep_last_row = [&]() {
        const int64_t rr = a.x_shared ? 0 : r;
        for (int j = lane; j < d; j += kWave) a.xlast[rr * d + j] = xg[(int64_t)(n - 1) * d + j];
        if (lane == 0) a.x2last[rr] = whole_x2[n - 1];
    };

    const V *row0 = reinterpret_cast<const V *>(ring);
    const float *yrow = a.y ? a.y + (int64_t)r * a.y_run_stride : nullptr;

    // Each role runs its own copy of the tile loop (same number of barriers in each), so
    // that the register-resident vector of one role never meets another role's code.
    if (!active) {
        for (int k = 0; k < ntiles; ++k) {
            if (k + 2 < ntiles) issue_tile(k + 2);
            if (WHOLE && OPT && k + 1 == ntiles && i == a.per_run) keep_last_row();
            tile_sync();
        }
        if (WHOLE) whole_meta<LOSS>(a, ring, r, i, lane, 0.f, 0.f, ws);
        return;
    }

    if (is_cmp) {
        // ---- comparator wavefront: z_t = <u_t, x_t>, no step -----------------------------
        float uv[NV][VW];
        auto load_u = [&](int sg) {
            const float *src = a.u + ((int64_t)r * a.S + sg) * d;
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    const int j = (m * kWave + lane) * VW + e;
                    uv[m][e] = j < d ? src[j] : 0.f;
                }
        };
        auto dot_u = [&](const V *xr) {
            float acc[VW];
#pragma unroll
            for (int e = 0; e < VW; ++e) acc[e] = 0.f;
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                float xv[VW];
                unpack<VW>(xr[m * kWave + lane], xv);
#pragma unroll
                for (int e = 0; e < VW; ++e) acc[e] = fmaf(uv[m][e], xv[e], acc[e]);
                if (NV > 4 && (m & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
            return wave_sum(combine<VW>(acc));
        };
        int seg = seg0;
        if (!WHOLE)
            while (seg + 1 < a.S && a.seg_start[seg + 1] <= a.t0) ++seg;
        int64_t next_seg = seg + 1 < a.S ? a.seg_start[seg + 1] : INT64_MAX;   // absolute round
        if constexpr (PRE) {
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) uv[m][e] = first[m][e];
        } else {
            load_u(seg);
        }
        float z = dot_u(row0), zreg = 0.f;
        float *zrow = a.Z + (int64_t)r * a.zl.zs_r + (int64_t)K * a.zl.zs_i;
        for (int k = 0; k < ntiles; ++k) {
            if (k + 2 < ntiles) issue_tile(k + 2);
            const int rmax = min(RT, n - k * RT);
            const float *rows = ring + (k % kRing) * TILE, *rows_next = ring + ((k + 1) % kRing) * TILE;
#pragma unroll 1
            for (int rr = 0; rr < rmax; ++rr) {
                const int t = k * RT + rr;
                if (lane == (t & 63)) zreg = z;
                if (a.t0 + t + 1 == next_seg) {     // the next round starts a new segment
                    ++seg;
                    next_seg = seg + 1 < a.S ? a.seg_start[seg + 1] : INT64_MAX;
                    load_u(seg);
                }
                z = dot_u(reinterpret_cast<const V *>(rr + 1 < RT ? rows + (rr + 1) * DP : rows_next));
                if (!WHOLE && ((t & 63) == 63 || t == n - 1)) {
                    const int tb = t & ~63;
                    if (tb + lane <= t) zrow[(int64_t)(tb + lane) * a.zl.zs_t] = zreg;
                }
            }
            tile_sync();
        }
        if (WHOLE) whole_meta<LOSS>(a, ring, r, i, lane, zreg, 0.f, ws);
        return;
    }

    // ---- learner wavefront ---------------------------------------------------------------
    auto dot_total = [](const float (&p)[VW]) {
        if constexpr (NACC == 4) return (p[0] + p[1]) + (p[2] + p[3]);
        else if constexpr (NACC == 2) return p[0] + p[1];
        else return p[0];
    };
    float wv[NV][VW];           // v = iterate / sigma
    float xa[NV][VW], xb[NV][VW];   // x_t / x_{t+1}, swapping roles every round
    float sigma = WHOLE ? sigma0 : a.sigma[(int64_t)r * K + i];
    float n2 = (float)(WHOLE ? n20 : a.n2[(int64_t)r * K + i]);  // ||v||^2 (kept as float64 in the state)
    const float eta = WHOLE ? eta0 : a.eta[i];
    float qv, z, zreg = 0.f, yreg = 0.f, x2reg = 0.f;   // qv = <v, x_t>, z = sigma qv
    // optimistic update: the hint is ha * x_{t-1}; hp = <w^_t, x_{t-1}>; g01 = <x_{t-1}, x_t>
    float ha = 0.f, hp = 0.f, x2prev = 0.f, g01reg = 0.f;
    if (OPT) {
        ha = WHOLE ? ha0 : a.ha[(int64_t)r * K + i];
        hp = WHOLE ? hp0 : a.hp[(int64_t)r * K + i];
        x2prev = WHOLE ? x2last0 : a.x2last[a.x_shared ? 0 : r];
    }
    {
        const float *src = a.V + ((int64_t)r * K + i) * d;
        float acc[VW];
#pragma unroll
        for (int e = 0; e < VW; ++e) acc[e] = 0.f;
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            unpack<VW>(row0[m * kWave + lane], xa[m]);
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                const int j = (m * kWave + lane) * VW + e;
                wv[m][e] = PRE ? first[PRE ? m : 0][e] : j < d ? src[j] : 0.f;
                acc[e & (NACC - 1)] = fmaf(wv[m][e], xa[m][e], acc[e & (NACC - 1)]);   // same order as the passes
                xb[m][e] = 0.f;
            }
        }
        qv = wave_sum(dot_total(acc));
        z = sigma * qv;                               // z_0 = <w_0, x_0>
    }
    const float *x2row = a.x2 + (a.x_shared ? 0 : (int64_t)r * a.x2_run_stride);
    const float *g01row = OPT ? a.g01 + (a.x_shared ? 0 : (int64_t)r * a.x2_run_stride) : nullptr;
    const int phase = (int)(a.t0 & 63);               // exact norms at absolute rounds = 63 mod 64

    const float D = a.D;
    const float D2 = D * D;
    float *zrow = a.Z + (int64_t)r * a.zl.zs_r + (int64_t)i * a.zl.zs_i;
    // sigma changes only when a projection is active (and only downwards): its reciprocal and
    // the threshold D^2 / sigma^2 on ||v||^2 are functions of sigma alone, recomputed with it,
    // so that a round that does not project pays one compare for the projection
    float isig = fast_rcp(sigma);
    float thr = D2 * isig * isig;
    const float eta2 = 2.0f * eta;

    // the pass over the registers: step and next-round dot
    auto pass = [&](float b, const V *xr, float (&xc)[NV][VW], float (&xn)[NV][VW], float (&aq)[VW]) {
#pragma unroll
        for (int e = 0; e < VW; ++e) aq[e] = 0.f;
#pragma unroll
        for (int j = 0; j < CH; ++j) unpack<VW>(xr[j * kWave + lane], xn[j]);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c + 1 < NCH) {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int m = (c + 1) * CH + j;
                    unpack<VW>(xr[m * kWave + lane], xn[m]);
                }
            }
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int m = c * CH + j;
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    const float w1 = fmaf(-b, xc[m][e], wv[m][e]);
                    wv[m][e] = w1;
                    aq[e & (NACC - 1)] = fmaf(w1, xn[m][e], aq[e & (NACC - 1)]);
                }
            }
            if (NCH > 2) __builtin_amdgcn_sched_barrier(0);
        }
    };

    // The same pass with one register set: chunk c of x_t is dead once the step has used it and
    // is refilled with chunk c of x_{t+1}; the dot runs kLag chunks behind so that the LDS
    // latency of the refill is covered.  Same operations in the same order as `pass`.
    auto pass_one = [&](float b, const V *xr, float (&xc)[NV][VW], float (&aq)[VW]) {
        if constexpr (kOneRowSet<NPL>) {
            static_assert(CH == 2 && VW == 4, "the ordering pin below lists the 8 values of a chunk");
            constexpr int kLag = 3;
            typedef float f4 __attribute__((ext_vector_type(4)));
            typedef const __attribute__((address_space(3))) f4 *LdsRow;
            LdsRow row = (LdsRow)(xr + lane);
#pragma unroll
            for (int e = 0; e < VW; ++e) aq[e] = 0.f;
#pragma unroll
            for (int c = 0; c < NCH + kLag; ++c) {
                if (c < NCH) {
                    const int m0 = c * CH;
#pragma unroll
                    for (int j = 0; j < CH; ++j)
#pragma unroll
                        for (int e = 0; e < VW; ++e) wv[m0 + j][e] = fmaf(-b, xc[m0 + j][e], wv[m0 + j][e]);
                    // the refill may only be issued once the step has read the old chunk: without
                    // this the LDS reads are hoisted to the top of the round (they do not depend
                    // on b) and both rows are live at once
                    asm volatile("" : "+v"(row)
                                 : "v"(wv[m0][0]), "v"(wv[m0][1]), "v"(wv[m0][2]), "v"(wv[m0][3]),
                                   "v"(wv[m0 + 1][0]), "v"(wv[m0 + 1][1]), "v"(wv[m0 + 1][2]), "v"(wv[m0 + 1][3]));
#pragma unroll
                    for (int j = 0; j < CH; ++j) {
                        const f4 fresh = row[(m0 + j) * kWave];
                        xc[m0 + j][0] = fresh.x; xc[m0 + j][1] = fresh.y;
                        xc[m0 + j][2] = fresh.z; xc[m0 + j][3] = fresh.w;
                    }
                }
                if (c >= kLag) {
#pragma unroll
                    for (int j = 0; j < CH; ++j) {
                        const int m = (c - kLag) * CH + j;
#pragma unroll
                        for (int e = 0; e < VW; ++e) aq[e & (NACC - 1)] = fmaf(wv[m][e], xc[m][e], aq[e & (NACC - 1)]);
                    }
                }
            }
        }
    };

    // Labels, ||x||^2 and <x_{t-1}, x_t> of the 64 rounds from t on, a lane each (t is a multiple of 64), and the
    // predictions of the rounds (t & ~63) .. t to Z: both happen at tile boundaries only (a tile's length divides
    // 64), so the tile loop does them and a round does not test for them.
    auto load_round_scalars = [&](int t) {
        if (WHOLE) {
            yreg = y0;
            x2reg = (lane < n) ? whole_x2[lane] : 0.f;
            if (OPT) g01reg = (lane < n) ? whole_x2[kWholeRounds + lane] : 0.f;
            return;
        }
        if (yrow) yreg = (t + lane < n) ? yrow[t + lane] : 0.f;
        x2reg = (t + lane < n) ? x2row[t + lane] : 0.f;
        if (OPT) g01reg = (t + lane < n) ? g01row[t + lane] : 0.f;
    };
    auto flush_predictions = [&](int t) {
        const int tb = t & ~63;
        if (tb + lane <= t && !WHOLE) zrow[(int64_t)(tb + lane) * a.zl.zs_t] = zreg;
    };
    // one round: consumes xc = x_t, fills xn = x_{t+1} from xnext; remeasure: ||v||^2 is summed afresh after the step
    auto round = [&](int t, const V *xnext, bool remeasure, float (&xc)[NV][VW], float (&xn)[NV][VW]) {
        const float yt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yreg), t & 63));
        const float x2t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x2reg), t & 63));
        // the prediction that is played and scored: plain, z = <w_t, x_t>; optimistic,
        // w_t = s (w^_t - ha x_{t-1}) with s from ||w^_t - ha x_{t-1}||^2, all from scalars
        float zp = z;
        if (OPT) {
            const float g01t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g01reg), t & 63));
            // ||w^_t - ha x_{t-1}||^2 in float32 like its inputs: it only matters where it exceeds D^2,
            // and there no term is much larger than the result
            const float mf = fmaf(ha * ha, x2prev, fmaf(-2.f * ha, hp, sigma * sigma * n2));
            const float sp = mf > D2 ? D * __builtin_amdgcn_rsqf(mf) : 1.f;
            zp = sp * fmaf(-ha, g01t, z);
        }
        if (lane == (t & 63)) zreg = zp;
        // fold sigma into v first (never between computing z and using it, so that z is
        // the same whether or not a call boundary falls here)
        if (sigma < kFoldLo) {                           // (sigma never grows: no upper test)
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) wv[m][e] *= sigma;
            n2 *= sigma * sigma;
            qv = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(z)));   // (uniform, like the sum it replaces)
            sigma = 1.f;
            isig = 1.f;
            thr = D2;
        }
        // w-space step along x_t; for the squared loss eta * 2 (z - y) = (2 eta) (z - y) exactly
        const float step = LOSS == 1 ? eta2 * (zp - yt) : eta * slope<LOSS>(zp, yt);
        const float b = step * isig;
        const float qold = qv;
        float aq[VW];
        if constexpr (kOneRowSet<NPL>) pass_one(b, xnext, xc, aq);
        else pass(b, xnext, xc, xn, aq);
        n2 = fmaxf(fmaf(b, fmaf(b, x2t, -2.f * qv), n2), 0.f);
        if (remeasure) {                                 // re-measure ||v||^2 exactly (replaces the identity's value)
            float an[VW];
#pragma unroll
            for (int e = 0; e < VW; ++e) an[e] = 0.f;
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) an[e] = fmaf(wv[m][e], wv[m][e], an[e]);
            n2 = wave_sum(combine<VW>(an));
        }
        qv = wave_sum(dot_total(aq));                      // <v, x_{t+1}>
        const float nrm = n2;                            // ||v||^2
        if (__builtin_amdgcn_ballot_w64(nrm > thr) != 0) {   // projection (the same in every lane)
            asm volatile("" ::: "memory");    // keeps the branch: its body is not to be run speculatively
            sigma = D * __builtin_amdgcn_rsqf(nrm);
            isig = fast_rcp(sigma);
            thr = D2 * isig * isig;
        }
        z = sigma * qv;
        if (OPT) {                                       // next round's hint and <w^_{t+1}, x_t>
            hp = sigma * fmaf(-b, x2t, qold);
            ha = step;
            x2prev = x2t;
        }
    };

    static_assert(64 % DenseCfg<NPL>::RT == 0, "tiles do not straddle the 64-round groups of labels and predictions");
    for (int k = 0; k < ntiles; ++k) {
        if (k + 2 < ntiles) issue_tile(k + 2);
        const int t0 = k * RT;
        const int rmax = min(RT, n - t0);
        if ((t0 & 63) == 0) load_round_scalars(t0);
        // rows of this tile follow one another in the ring; the row after its last is the next tile's first
        const float *rows = ring + (k % kRing) * TILE, *rows_next = ring + ((k + 1) % kRing) * TILE;
        const int rm = (63 - phase - t0) & 63;               // the round of this tile (if < RT) after which ||v||^2 is re-measured
        if constexpr (kOneRowSet<NPL>) {
#pragma unroll 1
            for (int rr = 0; rr < rmax; ++rr)
                round(t0 + rr, reinterpret_cast<const V *>(rr + 1 < RT ? rows + (rr + 1) * DP : rows_next), rr == rm, xa, xa);
        } else {
            if constexpr (kLoopOffset<NPL, LOSS> >= 0)
                asm volatile(".p2align 6\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"i"(kLoopOffset<NPL, LOSS>));
#pragma unroll 1
            for (int rr = 0; rr < rmax; rr += 2) {
                const int t = t0 + rr;
                round(t, reinterpret_cast<const V *>(rows + (rr + 1) * DP), rr == rm, xa, xb);          // (RT is even)
                if (rr + 1 < rmax)
                    round(t + 1, reinterpret_cast<const V *>(rr + 2 < RT ? rows + (rr + 2) * DP : rows_next), rr + 1 == rm, xb, xa);
            }
        }
        const int tl = t0 + rmax - 1;
        if ((tl & 63) == 63 || tl == n - 1) flush_predictions(tl);
        tile_sync();   // every wavefront has drained its copies: tile k+1 is complete; tile k may be overwritten
    }

    {
        float *dst = a.V + ((int64_t)r * K + i) * d;
#pragma unroll
        for (int m = 0; m < NV; ++m)
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                const int j = (m * kWave + lane) * VW + e;
                if (j < d) dst[j] = wv[m][e];
            }
        if (lane == 0) { a.sigma[(int64_t)r * K + i] = sigma; a.n2[(int64_t)r * K + i] = (double)n2; }
        if (OPT && lane == 0) { a.ha[(int64_t)r * K + i] = ha; a.hp[(int64_t)r * K + i] = hp; }
    }
    if (WHOLE) {
        whole_meta<LOSS>(a, ring, r, i, lane, zreg, yreg, ws);
        if (OPT && i == 0 && wpb == a.per_run) keep_last_row();
    }
}

}  // namespace
}  // namespace oco
