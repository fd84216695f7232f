// Dense rounds on the register kernel: the kernel with two learners per wavefront, the small kernels around
// the rounds, and how a call is enqueued.  The kernel itself: dense_rounds_kernel.h; short calls: dense_short.hip.
#include "dense_rounds_kernel.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>

namespace oco {
namespace {

constexpr int64_t kStreamPieceBytes = 64ll << 20;  // shared round stream per launch of a multi-pass grid
constexpr int64_t kPieceMinRounds = 512;           // no piece shorter than this
constexpr int64_t kBesideMaxWaves = 1024;          // one wavefront per SIMD: the chip is mostly idle
constexpr int64_t kBesidePieces = 4;
constexpr int64_t kHalfMinTasks = 8192;           // two learners per wavefront from this many learners on:
                                                   // four wavefronts per SIMD (with 4352 it measured 13 % slower)

// ---- two learners per wavefront ------------------------------------------------------------
// For d <= 1024 more than half of a round's instructions are its scalar section (slope, norm
// identity, reduction, projection), which every lane executes alike.  Here each half of a
// wavefront (32 lanes) owns one learner, so that section serves two learners at once; a lane
// keeps d/32 coordinates.  Shared round stream only; the comparators' predictions come from the
// contraction kernel, so every task is a learner.  Same arithmetic per learner as above except
// that sums run over 32 lanes.
template <int NPL> struct HalfCfg {
    static constexpr int RT = DenseCfg<NPL / 2>::RT;   // same tile bytes as the kernel above at equal d
    static constexpr int MAXW = NPL >= 32 ? 12 : 16;   // register budget
};

// Sum over the 32 lanes of each half of the wavefront (fixed order: xor-butterfly inside each row
// of 16 lanes, then row 1 += row 0 and row 3 += row 2); every lane gets the sum of its half.
__device__ __forceinline__ float half_sum(float v, bool upper)
{
    v += dpp_term<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
    v += dpp_term<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
    v += dpp_term<0x141, 0xF>(v);   // row_half_mirror
    v += dpp_term<0x140, 0xF>(v);   // row_mirror
    asm("s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 0"
        : "+v"(v));
    const float lo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31));
    const float hi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
    return upper ? hi : lo;
}

template <int NPL, int LOSS, bool OPT>
__global__ void __launch_bounds__(HalfCfg<NPL>::MAXW * kWave)
dense_rounds_half_kernel(const DenseArgs a)
{
    constexpr int LW = 32;                      // lanes per learner
    constexpr int VW = 4;
    constexpr int NV = NPL / VW;
    constexpr int DP = NPL * LW;                // padded dimension
    constexpr int RT = HalfCfg<NPL>::RT;
    constexpr int TILE = RT * DP;
    constexpr int RING_ROUNDS = kRing * RT;
    constexpr int NI = TILE / 4 / kWave;
    constexpr int CH = NV >= 2 ? 2 : 1;
    constexpr int NCH = NV / CH;
    static_assert(NPL % 4 == 0 && TILE % (4 * kWave) == 0 && RT % 2 == 0, "tile shape");
    using V = float4;

    extern __shared__ float4 smem4[];
    float *ring = reinterpret_cast<float *>(smem4);

    const int tid = threadIdx.x;
    const int nthreads = blockDim.x;
    const int wpb = nthreads >> 6;
    const int lane = tid & 63;
    const int ll = lane & (LW - 1);             // lane inside the half
    const bool upper = lane >= LW;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n;
    const int d = a.d;
    const int K = a.K;

    // task = learner (run r, index i); the upper half of the last wavefront may have none: it
    // then repeats the last task and stores nothing
    const int64_t ntask = (int64_t)a.R * K;
    const int64_t q0 = 2 * ((int64_t)blockIdx.x * wpb + wave);
    const bool active = q0 < ntask;             // per wavefront
    const int64_t qraw = q0 + (upper ? 1 : 0);
    const bool store = qraw < ntask;
    const int64_t q = store ? qraw : ntask - 1;
    const int r = (int)(q / K), i = (int)(q % K);
    const float *xg = a.x;

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

    for (int e = tid; e < kRing * TILE / 4; e += nthreads) smem4[e] = make_float4(0.f, 0.f, 0.f, 0.f);
    tile_sync();
    const int ntiles = (n + RT - 1) / RT;
    issue_tile(0);
    if (ntiles > 1) issue_tile(1);
    tile_sync();

    auto xrow = [&](int t) { return reinterpret_cast<const V *>(ring + (t % RING_ROUNDS) * DP); };

    if (!active) {
        for (int k = 0; k < ntiles; ++k) {
            if (k + 2 < ntiles) issue_tile(k + 2);
            tile_sync();
        }
        return;
    }

    const float *yrow = a.y ? a.y + (int64_t)r * a.y_run_stride : nullptr;
    float wv[NV][VW];
    float xa[NV][VW], xb[NV][VW];
    float sigma = a.sigma[(int64_t)r * K + i];
    float n2 = (float)a.n2[(int64_t)r * K + i];
    const float eta = a.eta[i];
    float qv, z, zreg = 0.f, yreg = 0.f, x2reg = 0.f;
    float ha = 0.f, hp = 0.f, x2prev = 0.f, g01reg = 0.f;
    if (OPT) {
        ha = a.ha[(int64_t)r * K + i];
        hp = a.hp[(int64_t)r * K + i];
        x2prev = a.x2last[0];
    }
    {
        const float *src = a.V + ((int64_t)r * K + i) * d;
        float acc[2] = {0.f, 0.f};
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            unpack<VW>(xrow(0)[m * LW + ll], xa[m]);
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                const int j = (m * LW + ll) * VW + e;
                wv[m][e] = j < d ? src[j] : 0.f;
                acc[e & 1] = fmaf(wv[m][e], xa[m][e], acc[e & 1]);     // same order as the passes
                xb[m][e] = 0.f;
            }
        }
        qv = half_sum(acc[0] + acc[1], upper);
        z = sigma * qv;
    }
    const float *x2row = a.x2;
    const float *g01row = OPT ? a.g01 : nullptr;
    const int phase = (int)(a.t0 & 63);
    const float D = a.D;
    const float D2 = D * D;
    float *zrow = a.Z + (int64_t)r * a.zl.zs_r + (int64_t)i * a.zl.zs_i;
    float isig = fast_rcp(sigma);
    float thr = D2 * isig * isig;
    const float eta2 = 2.0f * eta;

    auto pass = [&](float b, const V *xr, float (&xc)[NV][VW], float (&xn)[NV][VW], float (&aq)[2]) {
        aq[0] = aq[1] = 0.f;
#pragma unroll
        for (int j = 0; j < CH; ++j) unpack<VW>(xr[j * LW + ll], xn[j]);
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            if (c + 1 < NCH) {
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const int m = (c + 1) * CH + j;
                    unpack<VW>(xr[m * LW + ll], xn[m]);
                }
            }
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int m = c * CH + j;
#pragma unroll
                for (int e = 0; e < VW; ++e) {
                    const float w1 = fmaf(-b, xc[m][e], wv[m][e]);
                    wv[m][e] = w1;
                    aq[e & 1] = fmaf(w1, xn[m][e], aq[e & 1]);
                }
            }
            if (NCH > 2) __builtin_amdgcn_sched_barrier(0);
        }
    };

    auto round = [&](int t, float (&xc)[NV][VW], float (&xn)[NV][VW]) {
        if ((t & (LW - 1)) == 0 && yrow) yreg = (t + ll < n) ? yrow[t + ll] : 0.f;   // per half: the runs may differ
        if ((t & 63) == 0) {
            x2reg = (t + lane < n) ? x2row[t + lane] : 0.f;
            if (OPT) g01reg = (t + lane < n) ? g01row[t + lane] : 0.f;
        }
        const float ylo = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yreg), t & (LW - 1)));
        const float yhi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(yreg), LW + (t & (LW - 1))));
        const float yt = upper ? yhi : ylo;
        const float x2t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x2reg), t & 63));
        float zp = z;
        if (OPT) {
            const float g01t = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g01reg), t & 63));
            // ||w^_t - ha x_{t-1}||^2 in float32 like its inputs: it only matters where it exceeds D^2,
            // and there no term is much larger than the result
            const float mf = fmaf(ha * ha, x2prev, fmaf(-2.f * ha, hp, sigma * sigma * n2));
            const float sp = mf > D2 ? D * __builtin_amdgcn_rsqf(mf) : 1.f;
            zp = sp * fmaf(-ha, g01t, z);
        }
        if (ll == (t & (LW - 1))) zreg = zp;
        if (sigma < kFoldLo) {                           // per learner: the halves may differ
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) wv[m][e] *= sigma;
            n2 *= sigma * sigma;
            qv = z;
            sigma = 1.f;
            isig = 1.f;
            thr = D2;
        }
        const float step = LOSS == 1 ? eta2 * (zp - yt) : eta * slope<LOSS>(zp, yt);
        const float b = step * isig;
        const float qold = qv;
        float aq[2];
        pass(b, xrow(t + 1), xc, xn, aq);
        if (((phase + t) & 63) == 63) {                  // re-measure ||v||^2 exactly
            float an[2] = {0.f, 0.f};
#pragma unroll
            for (int m = 0; m < NV; ++m)
#pragma unroll
                for (int e = 0; e < VW; ++e) an[e & 1] = fmaf(wv[m][e], wv[m][e], an[e & 1]);
            n2 = half_sum(an[0] + an[1], upper);
        } else {
            n2 = fmaxf(fmaf(b, fmaf(b, x2t, -2.f * qv), n2), 0.f);
        }
        qv = half_sum(aq[0] + aq[1], upper);             // <v, x_{t+1}>
        const float nrm = n2;
        const bool pj = nrm > thr;                       // projection, per learner
        if (__builtin_amdgcn_ballot_w64(pj) != 0) {
            asm volatile("" ::: "memory");               // keeps the branch
            const float s2 = D * __builtin_amdgcn_rsqf(nrm);
            const float i2 = fast_rcp(s2);
            sigma = pj ? s2 : sigma;
            isig = pj ? i2 : isig;
            thr = pj ? D2 * i2 * i2 : thr;
        }
        z = sigma * qv;
        if (OPT) {
            hp = sigma * fmaf(-b, x2t, qold);
            ha = step;
            x2prev = x2t;
        }
        if ((t & (LW - 1)) == LW - 1 || t == n - 1) {    // flush the z of rounds (t & ~31) .. t
            const int tb = t & ~(LW - 1);
            if (tb + ll <= t && store) zrow[(int64_t)(tb + ll) * a.zl.zs_t] = zreg;
        }
    };

    for (int k = 0; k < ntiles; ++k) {
        if (k + 2 < ntiles) issue_tile(k + 2);
        const int rmax = min(RT, n - k * RT);
#pragma unroll 1
        for (int rr = 0; rr < rmax; rr += 2) {
            const int t = k * RT + rr;
            round(t, xa, xb);
            if (rr + 1 < rmax) round(t + 1, xb, xa);
        }
        tile_sync();
    }

    if (store) {
        float *dst = a.V + ((int64_t)r * K + i) * d;
#pragma unroll
        for (int m = 0; m < NV; ++m)
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                const int j = (m * LW + ll) * VW + e;
                if (j < d) dst[j] = wv[m][e];
            }
        if (ll == 0) { a.sigma[(int64_t)r * K + i] = sigma; a.n2[(int64_t)r * K + i] = (double)n2; }
        if (OPT && ll == 0) { a.ha[(int64_t)r * K + i] = ha; a.hp[(int64_t)r * K + i] = hp; }
    }
}

// ||x_t||^2 of every round row and, if g01 is given, <x_{t-1}, x_t> (x_{-1} = the last row of the
// previous call, kept in xlast): one wavefront per row, fixed summation order.
__global__ void __launch_bounds__(256) xnorm2_kernel(const float *x, int64_t run_stride, int nruns,
                                                     int n, int d, float *out, int64_t out_stride,
                                                     float *g01, const float *xlast)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= (int64_t)nruns * n) return;
    const int rr = (int)(row / n), t = (int)(row % n);
    const float *src = x + (int64_t)rr * run_stride + (int64_t)t * d;
    float x2, g = 0.f;
    row_scalars(src, g01 ? (t > 0 ? src - d : xlast + (int64_t)rr * d) : nullptr, d, lane, x2, g);
    if (lane == 0) {
        out[(int64_t)rr * out_stride + t] = x2;
        if (g01) g01[(int64_t)rr * out_stride + t] = g;
    }
}

// keeps the last round row of a call (and its squared norm) for the next call's hint terms
__global__ void __launch_bounds__(256) keep_last_row_kernel(const float *x, int64_t run_stride, int n, int d,
                                                            const float *x2, int64_t x2_stride, float *xlast,
                                                            float *x2last)
{
    const int rr = blockIdx.y;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < d) xlast[(int64_t)rr * d + j] = x[(int64_t)rr * run_stride + (int64_t)(n - 1) * d + j];
    if (j == 0) x2last[rr] = x2[(int64_t)rr * x2_stride + n - 1];
}

// Duration of one pass of the grid with l wavefronts on each SIMD, in units of a pass with one,
// fitted to sweeps on MI355X: up to about four wavefronts per SIMD mostly fill each other's
// stalls (the round is a dependent chain), beyond that they share the issue slots.
static double pass_cost(double l)
{
    return l <= 1.0 ? 1.0 : l <= 4.0 ? 1.0 + 0.1 * (l - 1.0) : l <= 6.0 ? 1.3 + 0.2 * (l - 4.0) : 1.7 + 0.55 * (l - 6.0);
}

// how one call's round kernel is launched: fixed for the call, used for each of its pieces
struct DensePlan {
    void (*kern)(const DenseArgs) = nullptr;
    size_t smem = 0;
    int wpb = 0;              // wavefronts per workgroup
    int rt = 0, rt0 = 0;      // rounds per tile of the ring, and the fewest (0: the kernel with two learners per wavefront)
    int64_t nwg = 0;          // workgroups
    int64_t batches = 0;      // passes the grid needs when the chip cannot hold it at once
    double cost = 0.0;        // modelled duration, in units of one lightly loaded pass
};

// Rounds per tile.  A tile is waited for at the end of the tile before it, so a tile has to last as long as a load
// from HBM takes (1 - 2 us) or every tile waits for the rest; the tiles of DenseCfg last that long only beside other
// wavefronts (two rounds of d = 1024: 1 us).  Where the grid leaves LDS idle -- `resident` workgroups per compute
// unit are all it needs -- tiles grow into it, to at most 32 rounds: no result depends on their length.
// Measured, streams of their own, 2000 rounds: 48 runs of 5 learners, d = 777 0.80 -> 0.68 us per round; 64 runs of 15,
// d = 1000 0.73 -> 0.53, d = 2048 1.01 -> 0.84; one run of 4, d = 1000 0.53 -> 0.41.
int tile_rounds(int rt, size_t round_bytes, int64_t resident)
{
    const size_t room = (size_t)(160 * 1024) / (size_t)std::max<int64_t>(1, resident);
    while (rt < 32 && kRing * 2 * (size_t)rt * round_bytes <= room) rt *= 2;
    return rt;
}

template <int NPL>
hipError_t plan_npl(const DenseArgs &a, int loss, DensePlan *plan)
{
    using C = DenseCfg<NPL>;
    const size_t smem = sizeof(float) * kRing * C::RT * NPL * kWave;
    void (*kern)(const DenseArgs) = nullptr;
    switch (loss * 2 + (a.optimistic ? 1 : 0)) {
        case 0: kern = dense_rounds_kernel<NPL, 0, false, false>; break;
        case 1: kern = dense_rounds_kernel<NPL, 0, true, false>; break;
        case 2: kern = dense_rounds_kernel<NPL, 1, false, false>; break;
        case 3: kern = dense_rounds_kernel<NPL, 1, true, false>; break;
        case 4: kern = dense_rounds_kernel<NPL, 2, false, false>; break;
        case 5: kern = dense_rounds_kernel<NPL, 2, true, false>; break;
        default: return hipErrorInvalidValue;
    }
    {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (ncu <= 0) ncu = 256;

    // Wavefronts per workgroup: the value that leaves the least work on the busiest compute
    // unit.  A unit gets ceil(nWG / ncu) workgroups, c of them resident at a time: so many full
    // passes plus a last, emptier one.  A pass puts l = resident*wpb/4 wavefronts on each SIMD
    // and its duration grows with l as g(l), fitted to sweeps on MI355X: up to about four
    // wavefronts per SIMD mostly fill each other's stalls (the round is a dependent chain),
    // beyond that they share the issue slots.
    const int per_run = a.per_run;
    int best = 0;
    double best_cost = 0.0;
    for (int w = C::MAXW; w >= 1; --w) {
        // A workgroup's wavefronts are dealt to the four SIMDs in turn and there is a barrier per
        // tile, so sizes that are not a multiple of four leave SIMDs unevenly loaded (measured up
        // to 20-60 % slower at equal occupancy): they pay a penalty and win only where they save a
        // pass of the grid.  Tiny workgroups only for tiny runs.
        if (w < 3 && !(per_run < 4 && w == per_run)) continue;
        int c = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, reinterpret_cast<const void *>(kern),
                                                         w * kWave, smem) != hipSuccess || c <= 0)
            continue;
        const int64_t nwg = a.x_shared ? ((int64_t)a.R * per_run + w - 1) / w
                                       : (int64_t)a.R * ((per_run + w - 1) / w);
        const int64_t per_cu = (nwg + ncu - 1) / ncu;
        const int64_t full = per_cu / c, rem = per_cu % c;
        double cost = (double)full * pass_cost((double)(c * w) / 4.0) + (rem ? pass_cost((double)(rem * w) / 4.0) : 0.0);
        if (w % 4 != 0 && per_run % w != 0) cost *= 1.1;
        // on equal cost prefer more, smaller workgroups per unit (fewer wavefronts held up by one
        // barrier), down to eight wavefronts (below that the per-workgroup staging of x shows)
        const bool better = best == 0 || cost < best_cost * (1.0 - 1e-9) ||
                            (w >= 8 && cost <= best_cost * (1.0 + 1e-9));
        if (better) { best = w; best_cost = cost; }
    }
    {                                                     // tuning choice: wavefronts per workgroup
        const int w = (int)a.tune->get(OCO_OPT_DENSE_WPB);
        if (w >= 1 && w <= C::MAXW) best = w;
    }
    if (best == 0) return hipErrorInvalidConfiguration;
    plan->cost = best_cost;
    if (a.tune->get(OCO_OPT_VERBOSE) == 1)
        fprintf(stderr, "dense plan: NPL %d per_run %d -> wpb %d cost %.3f\n", NPL, per_run, best, best_cost);
    int c = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, reinterpret_cast<const void *>(kern), best * kWave,
                                                     smem) != hipSuccess || c <= 0)
        c = 1;
    plan->kern = kern;
    plan->wpb = best;
    plan->nwg = a.x_shared ? ((int64_t)a.R * per_run + best - 1) / best
                           : (int64_t)a.R * ((per_run + best - 1) / best);
    const size_t round_bytes = sizeof(float) * NPL * kWave;
    plan->rt0 = C::RT;
    plan->rt = kGrowTiles<NPL> ? tile_rounds(C::RT, round_bytes, std::min<int64_t>(c, (plan->nwg + ncu - 1) / ncu)) : C::RT;
    plan->smem = kRing * plan->rt * round_bytes;
    plan->batches = ((plan->nwg + ncu - 1) / ncu + c - 1) / c;
    return hipSuccess;
}

// the same for the kernel with two learners per wavefront (shared stream, learners only)
template <int NPL>
hipError_t plan_half(const DenseArgs &a, int loss, DensePlan *plan)
{
    using C = HalfCfg<NPL>;
    const size_t smem = sizeof(float) * kRing * C::RT * NPL * 32;
    void (*kern)(const DenseArgs) = nullptr;
    switch (loss * 2 + (a.optimistic ? 1 : 0)) {
        case 0: kern = dense_rounds_half_kernel<NPL, 0, false>; break;
        case 1: kern = dense_rounds_half_kernel<NPL, 0, true>; break;
        case 2: kern = dense_rounds_half_kernel<NPL, 1, false>; break;
        case 3: kern = dense_rounds_half_kernel<NPL, 1, true>; break;
        case 4: kern = dense_rounds_half_kernel<NPL, 2, false>; break;
        case 5: kern = dense_rounds_half_kernel<NPL, 2, true>; break;
        default: return hipErrorInvalidValue;
    }
    if (smem > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
    }
    int dev = 0, ncu = 256;
    if (hipGetDevice(&dev) == hipSuccess)
        (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (ncu <= 0) ncu = 256;
    const int64_t nwaves = ((int64_t)a.R * a.K + 1) / 2;
    int best = 0, best_c = 1;
    double best_cost = 0.0;
    for (int w = C::MAXW; w >= 3; --w) {
        int c = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&c, reinterpret_cast<const void *>(kern),
                                                         w * kWave, smem) != hipSuccess || c <= 0)
            continue;
        const int64_t nwg = (nwaves + w - 1) / w;
        const int64_t per_cu = (nwg + ncu - 1) / ncu;
        const int64_t full = per_cu / c, rem = per_cu % c;
        double cost = (double)full * pass_cost((double)(c * w) / 4.0) + (rem ? pass_cost((double)(rem * w) / 4.0) : 0.0);
        if (w % 4 != 0) cost *= 1.1;
        const bool better = best == 0 || cost < best_cost * (1.0 - 1e-9) || (w >= 8 && cost <= best_cost * (1.0 + 1e-9));
        if (better) { best = w; best_cost = cost; best_c = c; }
    }
    {                                                     // tuning choice
        const int w = (int)a.tune->get(OCO_OPT_DENSE_WPB);
        if (w >= 1 && w <= C::MAXW) best = w;
    }
    if (best == 0) return hipErrorInvalidConfiguration;
    plan->kern = kern;
    plan->smem = smem;
    plan->wpb = best;
    plan->nwg = (nwaves + best - 1) / best;
    plan->batches = ((plan->nwg + ncu - 1) / ncu + best_c - 1) / best_c;
    plan->cost = best_cost;
    if (a.tune->get(OCO_OPT_VERBOSE) == 1)
        fprintf(stderr, "dense plan (two learners per wavefront): NPL %d -> wpb %d cost %.3f\n", NPL, best, best_cost);
    return hipSuccess;
}

hipError_t launch_piece(const DensePlan &p, const DenseArgs &a, hipStream_t s)
{
    const int per_run = a.per_run;
    dim3 grid;
    if (a.x_shared)
        grid = dim3((unsigned)p.nwg, 1, 1);
    else
        grid = dim3((unsigned)((per_run + p.wpb - 1) / p.wpb), (unsigned)a.R, 1);
    hipError_t e = clock_begin(a.clock, s, "dense_round_kernel");
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(p.kern, grid, dim3(p.wpb * kWave), p.smem, s, a);
    e = hipGetLastError();
    return e != hipSuccess ? e : clock_end(a.clock, s);
}

}  // namespace

bool dense_supported(int64_t d, int x_shared) { return d >= 1 && d <= (x_shared ? OCO_MAX_DENSE_D : 64 * kWave); }

// The scalars of the round rows that the hint terms of the optimistic update need, for the rounds of a.n
// (all runs): ||x_t||^2 into a.x2 and <x_{t-1}, x_t> into a.g01 (x_{-1}: the row kept from the call before).
hipError_t launch_hint_scalars(const DenseArgs &a, hipStream_t s)
{
    const int nruns = a.x_shared ? 1 : a.R;
    const int64_t xstride = a.x_shared ? 0 : a.x_run_stride;
    const int64_t rows = (int64_t)nruns * a.n;
    hipLaunchKernelGGL(xnorm2_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, a.x, xstride, nruns,
                       a.n, a.d, a.x2, a.x2_run_stride, a.g01, a.xlast);
    return hipGetLastError();
}

// ... and the last row of the call with its squared norm, kept for the next call (a.x2 filled as above)
hipError_t launch_keep_last_row(const DenseArgs &a, hipStream_t s)
{
    const int nruns = a.x_shared ? 1 : a.R;
    const int64_t xstride = a.x_shared ? 0 : a.x_run_stride;
    hipLaunchKernelGGL(keep_last_row_kernel, dim3((unsigned)((a.d + 255) / 256), (unsigned)nruns), dim3(256), 0, s,
                       a.x, xstride, a.n, a.d, a.x2, a.x2_run_stride, a.xlast, a.x2last);
    return hipGetLastError();
}

// One piece of a call: the squared norms of its rows, its round kernel, and the row kept for the
// next piece's hint terms.
static hipError_t launch_dense_piece(const DensePlan &plan, const DenseArgs &a, hipStream_t s)
{
    const int nruns = a.x_shared ? 1 : a.R;
    const int64_t xstride = a.x_shared ? 0 : a.x_run_stride;
    const int64_t rows = (int64_t)nruns * a.n;
    hipLaunchKernelGGL(xnorm2_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, a.x, xstride, nruns,
                       a.n, a.d, a.x2, a.x2_run_stride, a.optimistic ? a.g01 : nullptr,
                       a.optimistic ? a.xlast : nullptr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (a.per_run == a.K) {
        ComparatorGemmArgs g{};
        g.x = a.x; g.u = a.u; g.seg_start = a.seg_start; g.S = a.S; g.Z = a.Z; g.zl = a.zl;
        g.d = a.d; g.K = a.K; g.R = a.R; g.t0 = a.t0; g.n = a.n; g.vec_ok = a.vec_ok;
        e = launch_comparator_gemm(g, s);
        if (e != hipSuccess) return e;
    }
    e = launch_piece(plan, a, s);
    if (e != hipSuccess || !a.optimistic) return e;
    hipLaunchKernelGGL(keep_last_row_kernel, dim3((unsigned)((a.d + 255) / 256), (unsigned)nruns), dim3(256), 0, s,
                       a.x, xstride, a.n, a.d, a.x2, a.x2_run_stride, a.xlast, a.x2last);
    return hipGetLastError();
}

// Works out how the round kernel of this configuration is launched (kernel, workgroup size,
// who takes the comparators' predictions).
static hipError_t make_dense_plan(DenseArgs &a, int loss, DensePlan *out)
{
    const int npl = (a.d + kWave - 1) / kWave;
    auto make_plan = [&](DensePlan *plan) {
        if (npl <= 1) return plan_npl<1>(a, loss, plan);
        if (npl <= 2) return plan_npl<2>(a, loss, plan);
        if (npl <= 4) return plan_npl<4>(a, loss, plan);
        if (npl <= 8) return plan_npl<8>(a, loss, plan);
        if (npl <= 16) return plan_npl<16>(a, loss, plan);
        if (npl <= 32) return plan_npl<32>(a, loss, plan);
        if (npl <= 64) return plan_npl<64>(a, loss, plan);
        return hipErrorInvalidValue;
    };
    // Each run has one more wavefront task than learners, the comparator's, which only takes
    // inner products.  With a shared stream those are one contraction (U X^T per comparator
    // segment) that a kernel of its own does on the matrix cores: worth it where the round
    // kernel's grid gets cheaper without the extra tasks (fewer passes over the chip).
    DensePlan plan;
    a.per_run = a.K + 1;
    hipError_t e = make_plan(&plan);
    if (e != hipSuccess) return e;
    if (a.x_shared) {
        const int mode = (int)a.tune->get(OCO_OPT_COMPARATOR_GEMM);     // 0 never, 1 always
        DensePlan alt;
        a.per_run = a.K;
        e = make_plan(&alt);
        if (e != hipSuccess) return e;
        if (mode == 1 || (mode != 0 && alt.cost < plan.cost * 0.98)) plan = alt;
        else a.per_run = a.K + 1;
    }

    // Two learners per wavefront where a round is mostly its scalar section (d <= 1024) and the
    // grid is large enough to be bound by instruction issue rather than by the latency of a round.
    {
        bool half = a.x_shared && a.d > 96 && a.d <= 1024 && (int64_t)a.R * a.K >= kHalfMinTasks;
        const int hv = (int)a.tune->get(OCO_OPT_DENSE_HALF);          // 0 never, 1 wherever it can run
        if (hv >= 0) half = hv != 0 && a.x_shared && a.d <= 1024;
        if (half) {
            const int nplh = (a.d + 31) / 32;
            a.per_run = a.K;                                // comparators: contraction kernel
            if (nplh <= 4) e = plan_half<4>(a, loss, &plan);
            else if (nplh <= 8) e = plan_half<8>(a, loss, &plan);
            else if (nplh <= 16) e = plan_half<16>(a, loss, &plan);
            else e = plan_half<32>(a, loss, &plan);
            if (e != hipSuccess) return e;
        }
    }
    *out = plan;
    return hipSuccess;
}

hipError_t launch_dense_rounds(const DenseArgs &a0, int loss, hipStream_t s, const PieceHook *hook, bool *meta_done)
{
    if (a0.n <= 0) return hipSuccess;
    const bool split = dense_split_wanted(a0), run = !split && dense_run_wanted(a0);
    a0.plan->after_split = split || run;
    if (split) return launch_dense_split(a0, loss, s, hook);
    if (run) return launch_dense_run(a0, loss, s, hook);
    if (dense_window_wanted(a0)) return launch_dense_window(a0, loss, s, hook);
    if (a0.d > 64 * kWave) return hipErrorInvalidValue;
    DenseArgs a = a0;
    // the plan depends on the configuration and the tuning choices only: made once per state
    DensePlan plan;
    if (a.plan->valid) {
        plan.kern = reinterpret_cast<void (*)(const DenseArgs)>(const_cast<void *>(a.plan->kern));
        plan.smem = a.plan->smem; plan.wpb = a.plan->wpb; plan.nwg = a.plan->nwg;
        plan.rt = a.plan->rt; plan.rt0 = a.plan->rt0;
        plan.batches = a.plan->batches;
        a.per_run = a.plan->per_run;
    } else {
        hipError_t e = make_dense_plan(a, loss, &plan);
        if (e != hipSuccess) return e;
        a.plan->kern = reinterpret_cast<const void *>(plan.kern);
        a.plan->smem = plan.smem; a.plan->wpb = plan.wpb; a.plan->nwg = plan.nwg;
        a.plan->rt = plan.rt; a.plan->rt0 = plan.rt0;
        a.plan->batches = plan.batches; a.plan->per_run = a.per_run;
        a.plan->valid = true;
    }
    hipError_t e = hipSuccess;

    // A short call of few learners, as one kernel: 64 calls of 8 optimistic rounds with the combined model read back
    // after each (3 learners, d = 1000) 3.39 -> 1.18 ms; 32 calls, 16 runs of 8 learners: of 8 rounds, d = 10
    // 1.25 -> 0.44 ms, d = 4096 2.24 -> 1.45; of 64 rounds (the longest that a wavefront's lanes hold) 1.63 -> 0.92
    // and 4.32 -> 3.72.
    if (plan.rt0 > 0 && a.per_run == a.K + 1 && (int64_t)a.R * a.per_run <= kBesideMaxWaves &&
        a.tune->get(OCO_OPT_DENSE_WPB) < 0 && dense_short_supported(a)) {
        a.rt = plan.rt0;                             // no longer than the call (what the ring need not hold is not cleared)
        while (a.rt < a.n && 2 * a.rt <= plan.rt) a.rt *= 2;
        e = launch_dense_short(a, loss, s);
        *meta_done = e == hipSuccess;
        return e;
    }

    // Rounds give the same bits under any split of a call, so a call may go as several launches:
    //  - A grid that takes several passes over the chip has workgroups at unrelated positions of a
    //    shared round stream, whose footprint is then the whole stream: pieces of at most
    //    kStreamPieceBytes keep the stream of a piece in the last-level cache for every pass.
    //  - A grid that leaves most of the chip idle lets the caller's per-piece work (the hook) run
    //    beside the following pieces.
    int64_t pieces = 1;
    bool beside = false;
    if (plan.batches > 1 && a.x_shared) {
        const int64_t bytes = (int64_t)a.n * a.d * (int64_t)sizeof(float);
        pieces = (bytes + kStreamPieceBytes - 1) / kStreamPieceBytes;
    } else if (hook && plan.nwg * plan.wpb <= kBesideMaxWaves) {
        pieces = kBesidePieces;
        beside = true;
    }
    if (a.tune->get(OCO_OPT_DENSE_PIECES) >= 1) pieces = a.tune->get(OCO_OPT_DENSE_PIECES);   // tuning choice
    pieces = std::max<int64_t>(1, std::min<int64_t>(pieces, a.n / kPieceMinRounds));
    const int64_t step = (a.n / pieces + 63) / 64 * 64;
    for (int64_t off = 0; off < a.n; off += step) {
        const int64_t len = std::min<int64_t>(step, a.n - off);
        DenseArgs b = a;
        b.rt = plan.rt;
        b.x = a.x + off * a.d; b.t0 = a.t0 + off; b.n = (int)len;
        if (b.y) b.y = a.y + off;
        b.x2 = a.x2 + off;
        if (b.g01) b.g01 = a.g01 + off;
        b.Z = a.Z + off * a.zl.zs_t;
        e = launch_dense_piece(plan, b, s);
        if (e == hipSuccess && beside) e = hook->fn(hook->ctx, (int)off, (int)len);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace oco
