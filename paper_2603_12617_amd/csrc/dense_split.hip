// Dense rounds of a few base learners of a wide model on a shared round stream: the windows of
// dense_window.hip with the coordinates of a tile of 16 learners split over many workgroups.
//
// dense_window_kernel gives a tile (or two) of learners to one workgroup for a whole launch.  With few
// learners that leaves the chip empty: 16 learners of d = 32768 are one workgroup on 256 compute units and a
// window of 64 rounds takes 940 us, nearly all of it one compute unit's matrix instructions and loads.  Here
// a window is ONE launch in which workgroup (tile, chunk) owns a range of the tile's coordinates:
//   (1) it sums the chunks' shares of W X_k^T that the launch before left (fixed order, float64),
//   (2) runs the 64 dependent rounds of its tile (chain_rounds) on four wavefronts, four learners each -- every chunk of
//       a tile repeats them from the same inputs, which costs nothing on compute units that would idle and saves a
//       second launch per window --, while the other four wavefronts fetch the operands of (3),
//   (3) applies the window's step to its coordinates, W <- F W - Bm X_k, and takes its share of
//       W X_{k+1}^T and of ||W||^2 of the new iterates for the launch after.
// The launch boundary is the only synchronisation between workgroups: what a launch reads of other
// workgroups' work (shares, hint scalars) it reads from one of two buffers and writes the other.  The inner
// products are those of the iterates themselves (no cross-Gram correction as in dense_window_kernel) and
// ||w||^2 is measured every window.
// What bounds it (wall clock per window; 256 learners of d = 2048, optimistic, logistic / 16 learners of d = 32768, plain,
// squared): the dependent rounds 8.4 / 3.9 us (on one wavefront, a quad of lanes per learner, 11.1 / 8.2), the sum over the chunks'
// shares and the other inputs in front of them 3 (16 chunks) / 6.3 (64: 26 bytes a clock, as many as a compute unit gets from
// L2; touching the lines beforehand gives nothing), the sweep 2.2 / 4.3 and the loads of half of its blocks
// behind the rounds 0.4 / 3, start and end of a launch 3.  4000 rounds of the first take 1.30 ms (1.48) against 3.0 ms on the
// register kernel; 2000 rounds of the second (64 chunks of 512 coordinates) 0.93 ms (1.13) against 29.4 ms on dense_window_kernel.
// (A chunk's range of blocks comes with the arguments and its place from the grid, a learner's run from a multiplication: two 64-bit divisions stood 0.7 us before
// the first load.)
//
// The round rows are read as they are, without the re-tiled copies of dense_window.hip: with few tiles
// a copy would cost more than it saves.  The Gram matrices of the windows are taken by
// split_gram_kernel, depth-split as well, from the same rows.
#include "dense_chain.h"
#include "../../include/oco.h"

#include <algorithm>
#include <cstdio>

namespace oco {
namespace {

constexpr int kSW = 8;                        // wavefronts per workgroup: all sweep, the first four run the dependent rounds before
constexpr int kPre = 4;                       // blocks of 16 coordinates a wavefront fetches in front of (beside) the dependent rounds
constexpr int kSplitMaxTiles = 128;           // two chunks each on 256 compute units (beyond: dense_window_kernel, two tiles per workgroup)
constexpr int kHookRounds = 256;              // rounds whose meta work goes beside the following windows (one tile of the meta kernel; the last are on their own)
constexpr int kShareFloats = kB * kM + kM;    // a chunk's share of W X^T, then of ||W||^2

struct LdsS {
    static constexpr int gd = 0;
    static constexpr int scal = gd + kGramBytes;
    static constexpr int yb = scal + kScalBytes;
    static constexpr int zb = yb + kYBytes;
    static constexpr int bm = zb + kYBytes;
    static constexpr int fv = bm + kBmBytes;
    static constexpr int q0 = fv + kM * 4;
    static constexpr int rec = q0 + kQBytes;
    static constexpr int n2 = rec + kQBytes;                       // float [kSW][4][16]: shares of ||w||^2
    static constexpr int total = n2 + kSW * 4 * kM * 4;
    // once the dependent rounds are done the Gram table's space holds the wavefronts' shares of W X^T
    static constexpr int part = gd;
};
static_assert(LdsS::part + kSW * kB * kM * 4 <= LdsS::scal, "shares in the Gram table's space");

// where the comparators' predictions of a window lie in its Gram matrix, below the diagonal: four blocks of 16 rounds of up to 16 runs
__device__ __forceinline__ int cmp_at(int run, int t) { return ((t < 16 ? 2 : 3) * 16 + run) * kB + (t < 16 ? t : t - 16); }

struct SplitArgs {
    WinPlanD plan;
    int wu;                  // window whose rounds and step this launch works; -1: none (the call's first launch)
    int chunks;              // workgroups per tile
    int per, more;           // depth blocks of a chunk, and how many chunks have one more
    unsigned per_run;        // 2^31 / K, rounded up: a learner's run without a division (exact while q K < 2^31)
    __device__ __forceinline__ int run_of(int q) const { return (int)(((uint64_t)(unsigned)q * per_run) >> 31); }
    const float *gram;       // of window wu
    int cmp;                 // ... with the comparators' predictions in it
    const float *pin;        // shares of W X_wu^T and ||W||^2, [tile][chunk][kShareFloats]
    float *pout;             // ... of W X_{wu+1}^T
    const float *ha_in, *hp_in;   // [R K]: the hint scalars before window wu
    float *ha_out, *hp_out;
};

// A block of the sweep as a wavefront holds it: 16 coordinates of 16 learners (lane: 4 coordinates of one
// learner), the rows of window wu in the order of (3) and those of window wu + 1 in the order of (1).
struct SplitBlock { f4 v; float xu[16]; f4 xq[4]; };

template <int LOSS, bool OPT>
__global__ void __launch_bounds__(kSW *kWave) dense_split_kernel(const DenseArgs a, const SplitArgs sp)
{
    using Lds = LdsS;
    constexpr int NT = kSW * kWave;
    extern __shared__ __align__(16) char lds[];
    const int d = a.d, K = a.K, nq = a.R * K;
    const int chunk = (int)blockIdx.x, tile = (int)blockIdx.y;
    const int b_lo = chunk * sp.per + min(chunk, sp.more), b_hi = b_lo + sp.per + (chunk < sp.more ? 1 : 0);
    const int q_base = tile * kM;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const bool upd = sp.wu >= 0;                                    // uniform over the grid
    const bool do_q = sp.wu + 1 < sp.plan.count();
    const int wu_s = upd ? sp.plan.start(sp.wu) : 0, wu_l = upd ? sp.plan.len(sp.wu) : 0;
    const int wq_s = do_q ? sp.plan.start(sp.wu + 1) : 0, wq_l = do_q ? sp.plan.len(sp.wu + 1) : 0;

    // ---- inputs of the dependent rounds: scalars of the wavefronts that run them, the rest to LDS ----
    // (all loads are on their way before the first is waited for: with the scalars and the sum of ||w||^2 loaded
    // behind the barrier the rounds of 64 chunks started 3 us later)
    const int lc = 4 * wave + lk;                                   // wavefronts 0 .. 3, the learner whose rounds this lane runs
    double n2 = 0.0;
    float eta = 0.f;
    Hint hint{0.f, 0.f, 0.f};
    if (upd) {
        if (wave < kNP) {
            const int q = q_base + lc;
            if (q < nq) {
                eta = a.eta[q - sp.run_of(q) * K];
                if (OPT) {
                    hint.ha = sp.ha_in[q];
                    hint.hp = sp.hp_in[q];
                    hint.x2p = wu_s == 0 ? a.x2last[0] : a.x2[wu_s - 1];
                }
            }
        }
        constexpr int kGPer = kB * kB / NT;                         // rows wave, wave + 8, ... of G, a column per lane
        float gv[kGPer];
#pragma unroll
        for (int i = 0; i < kGPer; ++i) gv[i] = sp.gram[tid + i * NT];
        float yv[kB * kM / NT];
#pragma unroll
        for (int i = 0; i < kB * kM / NT; ++i) {
            const int q = q_base + wave + kSW * i;                  // a learner per wavefront, a round per lane
            yv[i] = (a.y && q < nq && lane < wu_l) ? a.y[(int64_t)sp.run_of(q) * a.y_run_stride + wu_s + lane] : 0.f;
        }
        // the chunks' shares, summed in chunk order
        const float *p0 = sp.pin + (int64_t)tile * sp.chunks * kShareFloats + tid * 2;
        double s0 = 0.0, s1 = 0.0;
        // (in batches whose loads are all on their way before the first is added)
        auto sum_shares = [&](int c0, auto batch, auto norms) __attribute__((always_inline)) {
            constexpr int U = decltype(batch)::value;
            constexpr bool N = decltype(norms)::value;              // ||w||^2 of the stored iterates as well
            const float *p = p0 + (int64_t)c0 * kShareFloats;
            const float *pn = sp.pin + ((int64_t)tile * sp.chunks + c0) * kShareFloats + kB * kM + (lc & (kM - 1));
            float2 v[U];
            float m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                v[u] = *reinterpret_cast<const float2 *>(p + u * kShareFloats);
                if (N) m[u] = pn[u * kShareFloats];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                s0 += (double)v[u].x;
                s1 += (double)v[u].y;
                if (N) n2 += (double)m[u];
            }
        };
        auto batches = [&](auto norms) __attribute__((always_inline)) {
            int c = 0;
            for (; c + 16 <= sp.chunks; c += 16) sum_shares(c, std::integral_constant<int, 16>{}, norms);
            if (c + 8 <= sp.chunks) {
                sum_shares(c, std::integral_constant<int, 8>{}, norms);
                c += 8;
            }
            switch (sp.chunks - c) {
                case 7: sum_shares(c, std::integral_constant<int, 7>{}, norms); break;
                case 6: sum_shares(c, std::integral_constant<int, 6>{}, norms); break;
                case 5: sum_shares(c, std::integral_constant<int, 5>{}, norms); break;
                case 4: sum_shares(c, std::integral_constant<int, 4>{}, norms); break;
                case 3: sum_shares(c, std::integral_constant<int, 3>{}, norms); break;
                case 2: sum_shares(c, std::integral_constant<int, 2>{}, norms); break;
                case 1: sum_shares(c, std::integral_constant<int, 1>{}, norms); break;
                default: break;
            }
        };
        if (wave < kNP) batches(std::true_type{});
        else batches(std::false_type{});
        double *q0d = reinterpret_cast<double *>(lds + Lds::q0);
        *reinterpret_cast<d2 *>(q0d + (tid >> 3) * kQStride + 2 * (tid & 7)) = d2{s0, s1};
        double *gd = reinterpret_cast<double *>(lds + Lds::gd);
        double *scal = reinterpret_cast<double *>(lds + Lds::scal);
#pragma unroll
        for (int i = 0; i < kGPer; ++i) put_gram(gd, scal, wave + kSW * i, lane, gv[i]);
        float *yb = reinterpret_cast<float *>(lds + Lds::yb);
#pragma unroll
        for (int i = 0; i < kB * kM / NT; ++i) {
            yb[(wave + kSW * i) * kYStride + lane] = yv[i];
        }
        if (OPT && tid < kB) scal[2 * tid + 1] = tid < wu_l ? (double)a.g01[wu_s + tid] : 0.0;
        __syncthreads();
    }

    // ---- the sweep's side -----------------------------------------------------------------------
    // Of 32 consecutive blocks the wavefronts without dependent rounds take the first sixteen, four each, which they fetch beside
    // the rounds; the others take theirs behind them.
    auto nth_block = [&](int i) __attribute__((always_inline)) {
        return b_lo + (i / kPre) * (kSW * kPre) + (wave < kNP ? kPre * kNP : 0) + i % kPre * kNP + (wave & (kNP - 1));
    };
    const int q_sw = q_base + lr;
    const bool q_ok = q_sw < nq;
    float *vrow = a.V + (int64_t)(q_ok ? q_sw : 0) * d + 4 * lk;
    const bool whole = (!upd || wu_l == kB) && (!do_q || wq_l == kB);
    auto fetch = [&](int blk, SplitBlock &o) __attribute__((always_inline)) {
        if (blk >= b_hi) return;                                    // uniform over the wavefront, as in step()
        const f4 zero = f4{0.f, 0.f, 0.f, 0.f};
        if (whole && blk * 16 + 16 <= d) {
            // nothing to leave out: scalar bases and one offset per lane (with a condition per load a block's addresses and masks
            // are 170 instructions, so 60; lanes without a learner read learner 0's row, see step())
            o.v = *reinterpret_cast<const f4 *>(vrow + blk * 16);
            if (upd) {
                const float *x = a.x + (int64_t)wu_s * d + blk * 16;
                const unsigned off = (unsigned)(lk * d + lr);
#pragma unroll
                for (int i = 0; i < 16; ++i) o.xu[i] = (x + (int64_t)(4 * i) * d)[off];
            }
            if (do_q) {
                const float *x = a.x + (int64_t)wq_s * d + blk * 16;
                const unsigned off = (unsigned)(lr * d + 4 * lk);
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) o.xq[rb] = *reinterpret_cast<const f4 *>(x + (int64_t)(16 * rb) * d + off);
            }
            return;
        }
        const bool in4 = blk * 16 + 4 * lk < d, in1 = blk * 16 + lr < d;
        o.v = in4 ? *reinterpret_cast<const f4 *>(vrow + blk * 16) : zero;
        if (upd) {
            const float *x = a.x + (int64_t)wu_s * d + blk * 16 + lr;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int t = 4 * i + lk;
                o.xu[i] = (in1 && t < wu_l) ? x[(int64_t)t * d] : 0.f;
            }
        }
        if (do_q) {
            const float *x = a.x + (int64_t)wq_s * d + blk * 16 + 4 * lk;
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const int t = 16 * rb + lr;
                o.xq[rb] = (in4 && t < wq_l) ? *reinterpret_cast<const f4 *>(x + (int64_t)t * d) : zero;
            }
        }
    };
    SplitBlock pre[kPre];
    if (upd && wave < kNP) {
        (void)chain_rounds<LOSS, Lds, OPT>(lds, 0, wave, lane, wu_l, eta, (double)a.D, 1.0, 1.0, n2, &hint);
        const int q = q_base + lc;
        if (OPT && chunk == 0 && q < nq && lr == 0) {
            sp.ha_out[q] = hint.ha;
            sp.hp_out[q] = hint.hp;
        }
    }
#pragma unroll
    for (int i = 0; i < kPre; ++i) fetch(nth_block(i), pre[i]);
    __syncthreads();

    if (upd && sp.cmp && chunk == 0 && tile == 0) {             // the comparators' predictions of the window
        for (int r = wave; r < a.R; r += kSW)
            if (lane < wu_l) a.Z[(int64_t)r * a.zl.zs_r + (int64_t)K * a.zl.zs_i + (int64_t)(wu_s + lane) * a.zl.zs_t] = sp.gram[cmp_at(r, lane)];
    }
    if (upd && chunk == 0) {                                        // the window's predictions
        const float *zb = reinterpret_cast<const float *>(lds + Lds::zb);
#pragma unroll
        for (int l = wave; l < kM; l += kSW) {
            const int q = q_base + l, r = sp.run_of(q);
            if (q < nq && lane < wu_l)
                a.Z[(int64_t)r * a.zl.zs_r + (int64_t)(q - r * K) * a.zl.zs_i + (int64_t)(wu_s + lane) * a.zl.zs_t] = zb[l * kYStride + lane];
        }
    }
    {
        float bmr[16];
        float F = 1.f;
        if (upd) {
            const float *bml = reinterpret_cast<const float *>(lds + Lds::bm);
#pragma unroll
            for (int i = 0; i < 16; ++i) bmr[i] = bml[(4 * i + lk) * kBmStride + lr];
            F = reinterpret_cast<const float *>(lds + Lds::fv)[lr];
        } else if (q_ok) {
            F = a.sigma[q_sw];                                      // the state's lazy scale goes into the iterates
        }
        f4 acc[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[rb] = f4{0.f, 0.f, 0.f, 0.f};
        float nn = 0.f;
        auto step = [&](int blk, SplitBlock &o) __attribute__((always_inline)) {
            if (blk >= b_hi) return;                                // uniform over the wavefront
            f4 vb;
#pragma unroll
            for (int r = 0; r < 4; ++r) vb[r] = q_ok ? o.v[r] * F : 0.f;
            if (upd) {
                f4 vo = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 16; i += 2) {
                    vb = __builtin_amdgcn_mfma_f32_16x16x4f32(o.xu[i], bmr[i], vb, 0, 0, 0);
                    vo = __builtin_amdgcn_mfma_f32_16x16x4f32(o.xu[i + 1], bmr[i + 1], vo, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) vb[r] += vo[r];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) nn = fmaf(vb[r], vb[r], nn);
            if (q_ok && blk * 16 + 4 * lk < d) *reinterpret_cast<f4 *>(vrow + blk * 16) = vb;
            if (do_q) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
                        acc[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.xq[rb][r], vb[r], acc[rb], 0, 0, 0);
            }
        };
#pragma unroll
        for (int i = 0; i < kPre; ++i) step(nth_block(i), pre[i]);
        for (int i = kPre, blk = nth_block(i); blk < b_hi; blk = nth_block(++i)) {
            fetch(blk, pre[0]);
            step(blk, pre[0]);
        }
        float *part = reinterpret_cast<float *>(lds + Lds::part) + wave * kB * kM;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[(rb * 16 + 4 * lk + r) * kM + lr] = acc[rb][r];
        reinterpret_cast<float *>(lds + Lds::n2)[(wave * 4 + lk) * kM + lr] = nn;
    }
    __syncthreads();
    float *po = sp.pout + ((int64_t)tile * sp.chunks + chunk) * kShareFloats;
    if (do_q) {
        const float *part = reinterpret_cast<const float *>(lds + Lds::part);
#pragma unroll
        for (int u = 0; u < kB * kM / NT; ++u) {
            const int e = tid + u * NT;
            double sum = 0.0;
#pragma unroll
            for (int v = 0; v < kSW; ++v) sum += (double)part[v * kB * kM + e];
            po[e] = (float)sum;
        }
    }
    if (tid < kM) {
        const float *n2s = reinterpret_cast<const float *>(lds + Lds::n2) + tid;
        double sum = 0.0;
#pragma unroll
        for (int i = 0; i < kSW * 4; ++i) sum += (double)n2s[i * kM];
        po[kB * kM + tid] = (float)sum;
    }
}

// State out after the last window: the iterates carry scale 1, their squared norms from the chunks' shares.
__global__ void __launch_bounds__(64) split_finish_kernel(const DenseArgs a, int chunks, const float *share, const float *ha, const float *hp)
{
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (q >= a.R * a.K) return;
    const float *pn = share + (int64_t)(q / kM) * chunks * kShareFloats + kB * kM + q % kM;
    double n2 = 0.0;
#pragma unroll 16
    for (int c = 0; c < chunks; ++c) n2 += (double)pn[(int64_t)c * kShareFloats];
    a.sigma[q] = 1.f;
    a.n2[q] = n2;
    if (a.optimistic) { a.ha[q] = ha[q]; a.hp[q] = hp[q]; }
}

// G = X_w X_w^T of window w0 + blockIdx.x over the depth blocks of chunk blockIdx.y, out[(window gridDim.y +
// chunk) 4096].  The dependent rounds of a window read G[t][t2] for t2 >= t only: of the sixteen 16 x 16 blocks
// the ten on and above the diagonal are taken, dealt to the four wavefronts, the others are left unwritten -- but for four that, with at
// most sixteen runs and one comparator segment, hold the comparators' predictions U X_w^T of the chunk (CMP; cmp_at), a block per wavefront
// from the rows it has anyway.  (In a kernel of their own they read the stream once more: 2000 rounds of d = 32768 and 4 runs 142 us beside the
// 99 of this kernel, before the first window, which waits for both; so 120.)
// Every wavefront reads the 64 rows (from L1 for three of the four), three depth blocks ahead of its matrix instructions.
// The sums of a depth block (16 products) are added up in float64: as one float32 chain over a chunk's depth (270 products
// at d = 516) their error was that of ||x||^2 in every projection, and the iterates of large steps had up to three times the
// register kernel's.
constexpr int kGramBlocks[4] = {3, 3, 2, 2};                        // of a wavefront, and where they lie (each reads all four groups of rows, so any deal does)
constexpr int kGramRow[4][3] = {{0, 0, 0}, {1, 1, 1}, {2, 0, 0}, {3, 2, 0}};
constexpr int kGramCol[4][3] = {{0, 1, 2}, {1, 2, 3}, {2, 3, 0}, {3, 3, 0}};
template <bool CMP>
__global__ void __launch_bounds__(256) split_gram_kernel(const float *x, const float *u, int runs, int d, WinPlanD plan, int w0, float *out)
{
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int w = w0 + (int)blockIdx.x, nblk = (d + 15) / 16;
    const int ws = plan.start(w), wl = plan.len(w);
    const int b_lo = (int)((int64_t)blockIdx.y * nblk / gridDim.y), b_hi = (int)((int64_t)(blockIdx.y + 1) * nblk / gridDim.y);
    const float *xr = x + (int64_t)ws * d + 4 * lk, *ur = u + (int64_t)(lr < runs ? lr : 0) * d + 4 * lk;
    struct Rows { f4 v[4], u; };
    auto fetch = [&](int blk, Rows &o) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int t = 16 * b + lr;
            const bool ok = t < wl && blk < b_hi && blk * 16 + 4 * lk < d;
            o.v[b] = ok ? *reinterpret_cast<const f4 *>(xr + (int64_t)t * d + blk * 16) : f4{0.f, 0.f, 0.f, 0.f};
        }
        if (CMP) o.u = (lr < runs && blk < b_hi && blk * 16 + 4 * lk < d) ? *reinterpret_cast<const f4 *>(ur + blk * 16) : f4{0.f, 0.f, 0.f, 0.f};
    };
    auto blocks = [&](auto wc) __attribute__((always_inline)) {
        constexpr int W = decltype(wc)::value, NG = kGramBlocks[W], N = NG + (CMP ? 1 : 0);
        f4 acc[N];
        Rows o[4];
        double tot[N][4];
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[b][r] = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) fetch(b_lo + i, o[i]);
        for (int blk = b_lo; blk < b_hi; blk += 4) {
            static_for<4>([&](auto ic) __attribute__((always_inline)) {   // (past b_hi: zeros)
                constexpr int i = decltype(ic)::value;
                fetch(blk + i + 3, o[(i + 3) & 3]);
#pragma unroll
                for (int b = 0; b < N; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
                static_for<4>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    static_for<NG>([&](auto bc) __attribute__((always_inline)) {
                        constexpr int b = decltype(bc)::value, ra = kGramRow[W][b], cb = kGramCol[W][b];
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(o[i].v[ra][r], o[i].v[cb][r], acc[b], 0, 0, 0);
                    });
                    if (CMP) acc[N - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(o[i].u[r], o[i].v[W][r], acc[N - 1], 0, 0, 0);
                });
#pragma unroll
                for (int b = 0; b < N; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) tot[b][r] += (double)acc[b][r];
            });
        }
        float *g = out + ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * kB * kB;
        static_for<NG>([&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value, ra = kGramRow[W][b], cb = kGramCol[W][b];
#pragma unroll
            for (int r = 0; r < 4; ++r) g[(ra * 16 + 4 * lk + r) * kB + cb * 16 + lr] = (float)tot[b][r];
        });
        if (CMP) {
#pragma unroll
            for (int r = 0; r < 4; ++r) g[cmp_at(4 * lk + r, 16 * W + lr)] = (float)tot[N - 1][r];
        }
    };
    if (wave == 0) blocks(std::integral_constant<int, 0>{});
    else if (wave == 1) blocks(std::integral_constant<int, 1>{});
    else if (wave == 2) blocks(std::integral_constant<int, 2>{});
    else blocks(std::integral_constant<int, 3>{});
}

// ... and the chunks' sum, in chunk order
__global__ void __launch_bounds__(256) split_gram_sum_kernel(const float *part, int chunks, float *gram)
{
    const int e = (int)(blockIdx.x & 15) * 256 + threadIdx.x;
    const int64_t w = blockIdx.x >> 4;
    double s = 0.0;
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) s += (double)part[(w * chunks + c) * kB * kB + e];
    gram[w * kB * kB + e] = (float)s;
}

// How a call is laid out in the windowed kernels' scratch: two buffers of shares and of hint scalars, the Gram
// matrices of `group` windows at a time and their partial sums.
struct SplitPlan {
    int tiles, chunks, gram_chunks, group;
    size_t share_floats, hint_floats;
    size_t cmp_off;          // where the comparator's partial sums start
    int cmp_chunks;
};
bool make_split_plan(const DenseArgs &a, SplitPlan *p)
{
    const int nblk = (a.d + 15) / 16;
    const int64_t nq = (int64_t)a.R * a.K;
    p->tiles = (int)((nq + kM - 1) / kM);
    if (p->tiles > kSplitMaxTiles) return false;
    // (everything that decides how a sum is grouped follows from the configuration, not from the call: calls
    // cut at multiples of 64 rounds then give the same bits)
    const int nwin = (int)std::min<int64_t>(a.n_max / kB + 2, 1 << 20);
    const size_t room = dense_window_scratch_floats(a.n_max, a.d);
    p->hint_floats = (size_t)(nq + 63) / 64 * 64;
    // as many chunks as the chip has compute units for; more than 64 (the sum over their shares takes 1.1 us per sixteen) only
    // while a wavefront has four blocks or more: 1000 rounds of d = 65536, 16 learners, 64 / 128 chunks 750 / 670 us.  (Rounded
    // down to a multiple of 8, 19 tiles of d = 40000 have 8 chunks, not 13: 1500 / 1114 us for 800 rounds.)
    p->chunks = std::max(1, std::min({std::max(64, nblk / (kSW * kPre)), 256 / p->tiles, (nblk + kSW - 1) / kSW}));
    // The meta work of every 256 rounds runs beside a window, a workgroup per run: two of this kernel's wavefronts fill the registers of
    // a SIMD, so a chunk whose compute unit has one waits for it (25 us; that window took 28 us instead of 16).  Fewer chunks leave those
    // compute units free, where that costs a wavefront at most one block more, and none beyond those it fetches beforehand: 256
    // learners of d = 2048 in 32 runs 16 -> 14 chunks, 4000 rounds 1430 -> 1297 us; 720 of d = 600 in 60 5 -> 4, 1256 -> 1104; but a fifth
    // block (240 of d = 8192 in 60) 841 -> 880.
    const int apart = (int)std::max<int64_t>(0, 256 - a.R) / p->tiles;
    auto depth = [&](int chunks) { return (nblk + chunks * kSW - 1) / (chunks * kSW); };
    if (apart >= 1 && apart < p->chunks && (depth(apart) == depth(p->chunks) || depth(apart) <= std::min(kPre, depth(p->chunks) + 1)))
        p->chunks = apart;
    for (;; --p->chunks) {
        p->share_floats = (size_t)p->tiles * p->chunks * kShareFloats;
        const size_t fixed = 2 * p->share_floats + 4 * p->hint_floats;
        const size_t one = (size_t)2 * kB * kB;                   // a Gram matrix and one partial of it
        if (fixed + one <= room) {
            const size_t wins = (room - fixed) / (kB * kB);       // Gram-sized pieces left
            const size_t all = (size_t)std::min(nwin, 256), per = wins / all;
            p->gram_chunks = per < 2 ? 1 : std::max(1, std::min({32, nblk / 16, (int)std::min<size_t>(32, per - 1)}));
            p->group = (int)std::min<size_t>(all, wins / (1 + p->gram_chunks));
            if (p->group >= 1) {
                // what is left takes the partial sums of the comparators' predictions, where their tiles
                // (64 runs x 64 rounds) are too few for the chip
                p->cmp_off = fixed + (size_t)p->group * (1 + p->gram_chunks) * kB * kB;
                const int64_t tiles = ((a.n_max + 63) / 64) * (((int64_t)a.R + 63) / 64);
                const int64_t fit = (int64_t)((room - p->cmp_off) / ((size_t)a.R * a.n_max));
                p->cmp_chunks = (int)std::max<int64_t>(1, std::min<int64_t>({512 / tiles, (int64_t)a.d / 512, fit, 64}));
                return true;
            }
        }
        if (p->chunks <= 1) return false;
    }
}

}  // namespace

bool dense_split_wanted(const DenseArgs &a)
{
    if (!a.x_shared || !a.vec_ok || !a.gram || !a.scaled || a.tune->get(OCO_OPT_DENSE_PATH) == 1) return false;
    const int64_t ropt = a.tune->get(OCO_OPT_WINDOW_RESIDENT);
    if (ropt != -1 && ropt != 5) return false;
    SplitPlan p;
    if (!make_split_plan(a, &p)) return false;
    // Measured per pass of 2048 squared-loss rounds, register kernel / this one, ms: d = 516 0.81 / 0.63 (4 learners) and 0.94 / 0.72
    // (2048); d = 1000 0.83 / 0.67 and 0.98 / 0.85; d = 4096 1.95 / 0.71 and, 1024 learners, 2.73 / 1.23; of 512 rounds, d = 516 0.26 /
    // 0.25 and 0.31 / 0.27, d = 1000 0.26 / 0.24 and 0.34 / 0.32 (512 learners 0.265 / 0.275, the one point that lost).  Against
    // dense_window_kernel: 640 rounds, d = 8192 2.50 / 0.31 (2 learners) and 2.60 / 0.69 (1024), d = 65536 28.7 / 4.5 (1024); 128
    // tiles (2048 learners, 2048 rounds), d = 520 0.82 / 0.74, d = 1000 1.11 / 0.85, d = 4096 3.5 / 1.8; 160 tiles, one chunk each, lost
    // (d = 2048 1.63 / 1.81, d = 520 0.89 / 0.93).  A call costs about 60 us here whatever its length, hence the least n; one
    // that need not come here (d <= 4096) stays with the register kernel, whose results no cut of the horizon changes.
    // The horizon's last call, which is as short as the cuts leave it, stays with the kernel of the calls before it: equal
    // calls and a rest give the bits of one call (cuts at multiples of 64).
    const bool rest = a.plan->after_split && a.t0 + a.n == a.T;
    return ropt == 5 || a.d > 64 * kWave || (a.d > 512 && (a.n >= 512 || rest) && a.tune->get(OCO_OPT_DENSE_PATH) < 0);
}

hipError_t launch_dense_split(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook)
{
    if (a.n <= 0) return hipSuccess;
    SplitPlan p;
    if (!make_split_plan(a, &p)) return hipErrorInvalidValue;
    const WinPlanD plan{a.t0, a.n};
    const int nwin = plan.count();
    float *share[2] = {a.gram, a.gram + p.share_floats};
    float *hint0 = share[1] + p.share_floats;
    float *gram = hint0 + 4 * p.hint_floats, *gpart = gram + (size_t)p.group * kB * kB;
    const bool beside = hook && hook->fn && hook->beside && a.n >= 512;
    ComparatorGemmArgs g{};
    g.x = a.x; g.u = a.u; g.seg_start = a.seg_start; g.S = a.S; g.Z = a.Z; g.zl = a.zl;
    g.d = a.d; g.K = a.K; g.R = a.R; g.t0 = a.t0; g.n = a.n; g.vec_ok = a.vec_ok;
    g.chunks = p.cmp_chunks; g.part = a.gram + p.cmp_off; g.fine = true;
    hipStream_t cs = s;
    const bool cmp = a.R <= 16 && a.S == 1;                         // the comparators' predictions come with the Gram matrices
    hipError_t e = beside ? hook->beside(hook->ctx, &cs) : hipSuccess;   // only the meta kernel reads its output
    if (e == hipSuccess && !cmp) e = launch_comparator_gemm(g, cs);
    if (e == hipSuccess && a.optimistic) e = launch_hint_scalars(a, s);
    if (e != hipSuccess) return e;
    void (*kern)(const DenseArgs, const SplitArgs) = nullptr;
    switch (loss * 2 + (a.optimistic ? 1 : 0)) {
        case 0: kern = dense_split_kernel<0, false>; break;
        case 1: kern = dense_split_kernel<0, true>; break;
        case 2: kern = dense_split_kernel<1, false>; break;
        case 3: kern = dense_split_kernel<1, true>; break;
        case 4: kern = dense_split_kernel<2, false>; break;
        case 5: kern = dense_split_kernel<2, true>; break;
        default: return hipErrorInvalidValue;
    }
    if (a.tune->get(OCO_OPT_VERBOSE) == 1)
        fprintf(stderr, "dense plan: windowed contraction kernel, %d windows, %d tiles in %d chunks of coordinates, Gram matrices of %d windows at a time in %d chunks\n",
                nwin, p.tiles, p.chunks, p.group, p.gram_chunks);
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LdsS::total);
    if (e != hipSuccess) return e;
    int done = 0;                                                   // rounds handed to the hook
    for (int w = -1; w < nwin; ++w) {
        const int in_group = w < 0 ? 0 : w % p.group;
        if (w >= 0 && in_group == 0) {
            const int nw = std::min(p.group, nwin - w);
            float *to = p.gram_chunks > 1 ? gpart : gram;
            if (cmp) hipLaunchKernelGGL(split_gram_kernel<true>, dim3((unsigned)nw, (unsigned)p.gram_chunks), dim3(256), 0, s, a.x, a.u, a.R, a.d, plan, w, to);
            else hipLaunchKernelGGL(split_gram_kernel<false>, dim3((unsigned)nw, (unsigned)p.gram_chunks), dim3(256), 0, s, a.x, a.x, 0, a.d, plan, w, to);
            if (p.gram_chunks > 1)
                hipLaunchKernelGGL(split_gram_sum_kernel, dim3((unsigned)nw * 16), dim3(256), 0, s, gpart, p.gram_chunks, gram);
        }
        SplitArgs sp{};
        sp.plan = plan; sp.wu = w; sp.chunks = p.chunks;
        const int nblk = (a.d + 15) / 16;
        sp.per = nblk / p.chunks; sp.more = nblk % p.chunks; sp.cmp = cmp;
        sp.per_run = (unsigned)((0x80000000u + (unsigned)a.K - 1) / (unsigned)a.K);
        sp.gram = gram + (size_t)in_group * kB * kB;
        sp.pin = share[w & 1]; sp.pout = share[(w + 1) & 1];
        float *hin = hint0 + (size_t)(w & 1) * 2 * p.hint_floats, *hout = hint0 + (size_t)((w + 1) & 1) * 2 * p.hint_floats;
        sp.ha_in = w == 0 ? a.ha : hin; sp.hp_in = w == 0 ? a.hp : hin + p.hint_floats;
        sp.ha_out = hout; sp.hp_out = hout + p.hint_floats;
        e = clock_begin(a.clock, s, "dense_split_kernel");
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)p.chunks, (unsigned)p.tiles), dim3(kSW * kWave), LdsS::total, s, a, sp);
        e = hipGetLastError();
        if (e == hipSuccess) e = clock_end(a.clock, s);
        if (e == hipSuccess && beside && w >= 0) {
            const int end = plan.start(w) + plan.len(w);
            if (w + 1 == nwin || end - done >= kHookRounds) {
                e = hook->fn(hook->ctx, done, end - done);
                done = end;
            }
        }
        if (e != hipSuccess) return e;
    }
    const int nq = a.R * a.K;
    const float *hl = hint0 + (size_t)(nwin & 1) * 2 * p.hint_floats;
    hipLaunchKernelGGL(split_finish_kernel, dim3((unsigned)((nq + 63) / 64)), dim3(64), 0, s, a, p.chunks, share[nwin & 1], hl, hl + p.hint_floats);
    e = hipGetLastError();
    if (e != hipSuccess || !a.optimistic) return e;
    return launch_keep_last_row(a, s);
}

}  // namespace oco
