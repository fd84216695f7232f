// Dense rounds of narrow models and of runs with a stream each: windows of 64 rounds, a tile of 16 learners of one stream per
// workgroup, everything a window needs inside it.
//
// The register kernel (dense_rounds_kernel.h) gives a wavefront to each learner; a round there is some 50 instructions and more
// of one wavefront, one after the other, and with few learners that is the whole time (64 runs of 15 learners, d = 100: 0.2 us per
// round; 48 of 5, d = 777, rows not aligned, optimistic: 0.65 us).  Here the rounds of a window are scalars of the window's Gram matrix
// (chain_rounds: 0.06 us per round, plain with the squared loss, whatever d is), and what grows with d is contractions on the
// matrix cores.  The stream is the workgroup's own (or all learners', few of them), so there is no pre-pass: no re-tiled copy of
// the rows and no Gram matrix in memory.  Window k:
//   (1) all wavefronts sum what the window before left in LDS, the shares of W X_k^T, in float64;
//   (2) wavefronts 0 .. 3 run the 64 dependent rounds, four learners each; wavefronts 4 .. 7 meanwhile take the Gram matrix of window
//       k + 1 and fetch the operands of their first blocks of (3);
//   (3) all apply the window's step to the iterates, W <- F W - Bm X_k, which stay in registers, block of 16 coordinates by block, and
//       take their shares of W X_{k+1}^T and ||W||^2.
// The rows are read as they are (any 4-byte address, any d), each three times from L2 (a compute unit draws about 20 bytes per clock from
// it: d = 777 400 KB and 8 us in (3)); a copy in LDS would be shared by one tile only.
// What bounds a window, wall clock: 64 runs of 15 learners, d = 100, plain, squared, 9.0 us (64 rounds on the register kernel 12.8): rounds
// 4.8 - 6 (3.9 with nothing beside them on their SIMD: the matrix instructions and float64 sums of the Gram matrix, 3.6 us, get in their
// way), (3) and the wait for it 2.1; 48 of 5, d = 777, optimistic, logistic, 26 us (41): rounds 15 (8 alone) beside a Gram matrix of 14, (3)
// 9.4; one learner of d = 10 5.5 us (10): rounds 3.4.  Per pass 2.30 -> 1.63 ms, 1.98 -> 1.43 ms, 0.250 -> 0.179 ms.
#include "dense_chain.h"
#include "../../include/oco.h"

#include <algorithm>
#include <cstdio>

namespace oco {
namespace {

constexpr int kRW = 8;                        // wavefronts per workgroup
constexpr int kRT = kRW * kWave;
// the ten 16 x 16 blocks of a Gram matrix on and above the diagonal, and dealt to wavefronts 4 .. 7 such that a wavefront needs two or three of the four groups of
// 16 rows (kGramNeeds)
constexpr int kGramParts = 10;
constexpr int kPartRow[kGramParts] = {0, 0, 0, 0, 1, 1, 1, 2, 2, 3}, kPartCol[kGramParts] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};
constexpr int kGramBlocks[4] = {3, 3, 2, 2};
constexpr int kGramRow[4][3] = {{0, 0, 0}, {1, 1, 1}, {2, 2, 0}, {0, 3, 0}};
constexpr int kGramCol[4][3] = {{0, 1, 2}, {1, 2, 3}, {2, 3, 0}, {3, 3, 0}};
constexpr bool kGramNeeds[4][4] = {{true, true, true, false}, {false, true, true, true}, {false, false, true, true}, {true, false, false, true}};
constexpr int kRunMaxBlocks = 16 * kRW;       // iterates of a tile in the registers of a workgroup: d <= 2048

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));   // four floats at any 4-byte address

// How a window's Gram matrix is taken: for narrow models (DEEP false) a few of its blocks per wavefront over the whole depth, straight
// into the table of the window, of which there are two; else the depth split over the wavefronts, whose shares meet in LDS, the rows read
// once.  (Blocks per wavefront read the rows two and a half times, from L1 while the window fits it: d = 777 18.5 us per window beside
// the rounds, split 11.)
template <bool DEEP> struct LdsR {
    static constexpr int tables = kGramBytes + kScalBytes;
    static constexpr int gd = 0;
    static constexpr int scal = gd + kGramBytes;
    static constexpr int yb = gd + (DEEP ? 1 : 2) * tables;
    static constexpr int zb = yb + kYBytes;
    static constexpr int bm = zb + kYBytes;
    static constexpr int fv = bm + kBmBytes;
    static constexpr int q0 = fv + kM * 4;
    static constexpr int n2 = q0 + kQBytes;                        // float [kRW][4][16]: shares of ||w||^2
    static constexpr int gpart = n2 + kRW * 4 * kM * 4;            // float [4][10][64][4]: shares of the Gram matrix
    static constexpr int part = gpart + (DEEP ? 4 * kGramParts * 1024 : 0);   // float [kRW][64][16]: shares of W X^T
    static constexpr int rec = part;                               // (what the rounds record: between the sum and the next shares)
    static constexpr int total = part + kRW * kB * kM * 4;
};
static_assert(LdsR<true>::total <= 160 * 1024 && LdsR<false>::total <= 160 * 1024 && kQBytes <= kRW * kB * kM * 4, "LDS of a gfx950 compute unit");

// the rows of a window for one block of 16 coordinates, in the lane order of (1) (round l % 16 of each of four groups, four
// coordinates) or of (3) (coordinate l % 16, rounds 4 i + l / 16)
struct RowsQ { f4 v[4]; };
struct RowsU { float v[16]; };
// no value, at no cost (left without one on some paths, the rows of the window before would be kept for them)
__device__ __forceinline__ void none(RowsQ &q, RowsU &u)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "=v"(q.v[i]));
#pragma unroll
    for (int i = 0; i < 16; ++i) asm volatile("" : "=v"(u.v[i]));
}

// The rows of a window through a buffer descriptor: one offset per lane and a scalar per block and group of rounds (added to it: the
// range check of a scalar offset beyond the range would wrap), and rounds past the call read as zero.  (A window that is shorter for another reason, the call's first, reads rounds of the one after: what they
// give is left out where the shares are summed, and Bm is zero there.)  Coordinates past d of the last block, which are the next
// row's first, are masked by who uses it.
struct Rows {
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ Rows(const float *xs, int d, const WinPlanD &plan, int w)
    {
        const int ws = plan.start(w), left = min(plan.n - ws, kB);
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(xs + (int64_t)ws * d), 0, left * d * 4, 0x00027000);
    }
    __device__ __forceinline__ f4 q1(int d, int off, int rb, int blk) const
    {
        return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + (rb * 16 * d + blk * 16) * 4, 0, 0));
    }
    __device__ __forceinline__ void q(int d, int off, int blk, RowsQ &o) const
    {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) o.v[rb] = q1(d, off, rb, blk);
    }
    __device__ __forceinline__ void u(int d, int off, int blk, RowsU &o) const
    {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            o.v[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off + (i * 4 * d + blk * 16) * 4, 0, 0));
    }
};

template <int LOSS, bool OPT, int NB>
__global__ void __launch_bounds__(kRT) dense_run_kernel(const DenseArgs a, WinPlanD plan, int w0, int nw, int per_tile)
{
    constexpr bool DEEP = NB > 2;
    using Lds = LdsR<DEEP>;
    extern __shared__ __align__(16) char lds[];
    const int K = a.K;
    // What a lane is and the row length, taken afresh in every phase of a window from values the compiler cannot see through: the many
    // addresses and scalar offsets that follow from them would otherwise be kept, and spilled, across the window loop.
    int d, tid, lane, lr, lk, wave, nfull, tail, offq, offu;
    auto afresh = [&]() __attribute__((always_inline)) {
        d = a.d;
        tid = (int)threadIdx.x;
        asm volatile("" : "+s"(d), "+v"(tid));
        lane = tid & 63;
        lr = lane & 15;
        lk = lane >> 4;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        nfull = d / 16;                                            // blocks of 16 coordinates
        tail = d & 15;                                             // coordinates of the last, partial one
        offq = (lr * d + 4 * lk) * 4;
        offu = (lk * d + lr) * 4;
    };
    afresh();
    // the tile's learners: of a shared stream any per_tile of all, of a stream of its own per_tile of that run's
    const int run = a.x_shared ? 0 : (int)blockIdx.y;
    const int q_lo = run * K + (int)blockIdx.x * per_tile;
    const int q_hi = min(q_lo + per_tile, a.x_shared ? a.R * K : run * K + K);
    const float *xs = a.x + (int64_t)run * (a.x_shared ? 0 : a.x_run_stride);
    const int64_t scal_off = a.x_shared ? 0 : (int64_t)run * a.x2_run_stride;

    // The b-th block a wavefront keeps: few blocks to wavefronts 4 .. 7 alone, which fetch their rows beside the dependent rounds.
    auto nth_block = [&](int b) __attribute__((always_inline)) {
        if (nfull <= kRW) return wave >= 4 ? wave - 4 + 4 * b : 1 << 20;
        return ((wave + 4) & 7) + kRW * b;
    };
    auto has_tail = [&]() __attribute__((always_inline)) { return tail != 0 && wave == 4 + (nfull & 3); };
    auto tail_in = [&](int r) __attribute__((always_inline)) { return 4 * lk + r < tail; };   // this lane's coordinates of the partial block
    auto mask_q = [&](RowsQ &x) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) x.v[rb][r] = tail_in(r) ? x.v[rb][r] : 0.f;
    };
    // inputs of the dependent rounds on their way: labels and (optimistic update) <x_{t-1}, x_t>
    struct Inputs { float y[2], hg, x2p; };                       // (x2p: ||x||^2 of the round before the window)
    auto load_inputs = [&](int w, Inputs &in) __attribute__((always_inline)) {
        const int ws = plan.start(w), wl = plan.len(w);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = q_lo + wave + kRW * i;
            in.y[i] = (a.y && q < q_hi && lane < wl) ? a.y[(int64_t)(q / K) * a.y_run_stride + ws + lane] : 0.f;
        }
        in.hg = (OPT && wave == 0 && lane < wl) ? a.g01[scal_off + ws + lane] : 0.f;
        in.x2p = !OPT ? 0.f : ws == 0 ? a.x2last[run] : a.x2[scal_off + ws - 1];
    };
    auto store_inputs = [&](const Inputs &in, int tab) __attribute__((always_inline)) {
        float *yb = reinterpret_cast<float *>(lds + Lds::yb);
#pragma unroll
        for (int i = 0; i < 2; ++i) yb[(wave + kRW * i) * kYStride + lane] = in.y[i];
        if (OPT && wave == 0) reinterpret_cast<double *>(lds + Lds::scal + tab)[2 * lane + 1] = (double)in.hg;
    };
    // a window's Gram matrix to LDS, sums of 16 products added up in float64: the blocks of this wavefront
    auto gram_blocks = [&](const Rows &rows, int wl, int tab) __attribute__((always_inline)) {
        double *gd = reinterpret_cast<double *>(lds + Lds::gd + tab), *scal = reinterpret_cast<double *>(lds + Lds::scal + tab);
        const int nblk = nfull + (tail != 0 ? 1 : 0);
        auto blocks = [&](auto wc) __attribute__((always_inline)) {
            constexpr int W = decltype(wc)::value, N = kGramBlocks[W];
            auto load = [&](int blk, RowsQ &o) __attribute__((always_inline)) {   // (past the last block: rounds or zeros that are not used)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
                    if (kGramNeeds[W][rb]) o.v[rb] = rows.q1(d, offq, rb, blk);
            };
            double tot[N][4];
#pragma unroll
            for (int b = 0; b < N; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) tot[b][r] = 0.0;
            RowsQ x[4];
#pragma unroll
            for (int i = 0; i < 3; ++i) load(i, x[i]);
            for (int blk = 0; blk < nblk; blk += 4) {
                static_for<4>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    load(blk + i + 3, x[(i + 3) & 3]);
                    if (blk + i < nblk) {
                        if (blk + i == nfull) mask_q(x[i]);
                        f4 acc[N];
#pragma unroll
                        for (int b = 0; b < N; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
                        static_for<4>([&](auto rc) __attribute__((always_inline)) {
                            constexpr int r = decltype(rc)::value;
                            static_for<N>([&](auto bc) __attribute__((always_inline)) {
                                constexpr int b = decltype(bc)::value, ra = kGramRow[W][b], cb = kGramCol[W][b];
                                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i].v[ra][r], x[i].v[cb][r], acc[b], 0, 0, 0);
                            });
                        });
#pragma unroll
                        for (int b = 0; b < N; ++b)
#pragma unroll
                            for (int r = 0; r < 4; ++r) tot[b][r] += (double)acc[b][r];
                    }
                });
            }
            static_for<N>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value, ra = kGramRow[W][b], cb = kGramCol[W][b];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int t = 16 * ra + 4 * lk + r, t2 = 16 * cb + lr;
                    put_gram(gd, scal, t, t2, t < wl && t2 < wl ? tot[b][r] : 0.0);
                }
            });
        };
        if (wave == 4) blocks(std::integral_constant<int, 0>{});
        else if (wave == 5) blocks(std::integral_constant<int, 1>{});
        else if (wave == 6) blocks(std::integral_constant<int, 2>{});
        else blocks(std::integral_constant<int, 3>{});
    };
    // ... or this wavefront's share of all of them, coordinate blocks wave - 4, wave, ...
    auto gram_share = [&](const Rows &rows) __attribute__((always_inline)) {
        double tot[kGramParts][4];
#pragma unroll
        for (int b = 0; b < kGramParts; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[b][r] = 0.0;
        const int nblk = nfull + (tail != 0 ? 1 : 0);
        constexpr int AHEAD = NB > 8 ? 2 : 4;                      // register sets of rows
        RowsQ x[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD - 1; ++i) rows.q(d, offq, wave - 4 + 4 * i, x[i]);
        for (int blk0 = wave - 4; blk0 < nblk; blk0 += 4 * AHEAD) {
            static_for<AHEAD>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                const int blk = blk0 + 4 * i;
                rows.q(d, offq, blk + 4 * (AHEAD - 1), x[(i + AHEAD - 1) % AHEAD]);
                if (blk < nblk) {
                    if (blk == nfull) mask_q(x[i]);
                    f4 acc[kGramParts];
#pragma unroll
                    for (int b = 0; b < kGramParts; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
                    static_for<4>([&](auto rc) __attribute__((always_inline)) {
                        constexpr int r = decltype(rc)::value;
                        static_for<kGramParts>([&](auto bc) __attribute__((always_inline)) {
                            constexpr int b = decltype(bc)::value;
                            acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i].v[kPartRow[b]][r], x[i].v[kPartCol[b]][r], acc[b], 0, 0, 0);
                        });
                    });
#pragma unroll
                    for (int b = 0; b < kGramParts; ++b) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) tot[b][r] += (double)acc[b][r];
                        if (b & 1) __builtin_amdgcn_sched_barrier(0);   // (all forty converted first would be eighty registers)
                    }
                }
            });
        }
        f4 *gp = reinterpret_cast<f4 *>(lds + Lds::gpart) + (wave - 4) * kGramParts * 64 + lane;
#pragma unroll
        for (int b = 0; b < kGramParts; ++b) gp[b * 64] = f4{(float)tot[b][0], (float)tot[b][1], (float)tot[b][2], (float)tot[b][3]};
    };
    auto sum_gram_shares = [&](int wl) __attribute__((always_inline)) {
        const f4 *gp = reinterpret_cast<const f4 *>(lds + Lds::gpart) + lane;
        double *gd = reinterpret_cast<double *>(lds + Lds::gd), *scal = reinterpret_cast<double *>(lds + Lds::scal);
        for (int b = wave; b < kGramParts; b += kRW) {
            double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const f4 g = gp[(v * kGramParts + b) * 64];
#pragma unroll
                for (int r = 0; r < 4; ++r) s[r] += (double)g[r];
            }
            const int ra = b < 4 ? 0 : b < 7 ? 1 : b < 9 ? 2 : 3, cb = b < 4 ? b : b < 7 ? b - 3 : b < 9 ? b - 5 : 3;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = 16 * ra + 4 * lk + r, t2 = 16 * cb + lr;
                put_gram(gd, scal, t, t2, t < wl && t2 < wl ? s[r] : 0.0);
            }
        }
    };
    auto gram = [&](const Rows &rows, int wl, int tab) __attribute__((always_inline)) {
        if constexpr (DEEP) gram_share(rows);
        else gram_blocks(rows, wl, tab);
    };
    auto put_share = [&](const f4 (&acc)[4]) __attribute__((always_inline)) {
        float *part = reinterpret_cast<float *>(lds + Lds::part) + wave * kB * kM;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[(rb * 16 + 4 * lk + r) * kM + lr] = acc[rb][r];
    };
    auto q_of = [&](const RowsQ &x, const f4 &v, f4 (&acc)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) acc[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[rb][r], v[r], acc[rb], 0, 0, 0);
    };
    // ||w||^2 of the learner whose rounds this lane runs, as the last sweep measured it: 32 shares, dealt to its 16 lanes
    auto measured_n2 = [&](int lc) __attribute__((always_inline)) {
        const float *n2s = reinterpret_cast<const float *>(lds + Lds::n2);
        return row_sum((double)n2s[lr * kM + lc] + (double)n2s[(16 + lr) * kM + lc]);
    };

    // ---- state in, and the shares of the first window -------------------------------------------
    const int q_ch = q_lo + 4 * wave + lk;                         // wavefronts 0 .. 3: the learner whose rounds this lane runs
    float eta = 0.f;
    double scale = 1.0, n2 = 0.0;
    Hint hint{0.f, 0.f, 0.f};
    if (wave < 4 && q_ch < q_hi) {
        eta = a.eta[q_ch % K];
        scale = (double)a.sigma[q_ch];
        n2 = a.n2[q_ch] * scale * scale;
        if (OPT) {
            hint.ha = a.ha[q_ch];
            hint.hp = a.hp[q_ch];
        }
    }
    const bool q_ok = q_lo + lr < q_hi;                            // this lane's learner in the sweep
    float *vrow = a.V + (int64_t)(q_ok ? q_lo + lr : q_lo) * d + 4 * lk;
    f4 V[NB + 1];                                                  // the tile's iterates: 4 coordinates of one learner per block; the partial one last
    static_for<NB>([&](auto bc) __attribute__((always_inline)) {
        constexpr int b = decltype(bc)::value;
        const int blk = nth_block(b);
        V[b] = f4{0.f, 0.f, 0.f, 0.f};
        if (blk < nfull && q_ok) V[b] = *reinterpret_cast<const f4u *>(vrow + blk * 16);
    });
#pragma unroll
    for (int r = 0; r < 4; ++r) V[NB][r] = (has_tail() && q_ok && tail_in(r)) ? vrow[nfull * 16 + r] : 0.f;
    Inputs in;
    load_inputs(w0, in);
    {
        const Rows rows(xs, d, plan, w0);
        f4 acc[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[rb] = f4{0.f, 0.f, 0.f, 0.f};
        static_for<NB>([&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value;
            const int blk = nth_block(b);
            if (blk < nfull) {
                RowsQ x;
                rows.q(d, offq, blk, x);
                q_of(x, V[b], acc);
            }
        });
        if (has_tail()) {
            RowsQ x;
            rows.q(d, offq, nfull, x);
            mask_q(x);
            q_of(x, V[NB], acc);
        }
        put_share(acc);
        if (wave >= 4) gram(rows, plan.len(w0), DEEP ? 0 : (w0 & 1) * Lds::tables);
    }
#pragma unroll 1
    for (int k = 0; k < nw; ++k) {
        afresh();
        const int w = w0 + k, wl = plan.len(w);
        const bool more = k + 1 < nw;
        const int tab = DEEP ? 0 : (w & 1) * Lds::tables;
        const Rows rows(xs, d, plan, w), ahead(xs, d, plan, more ? w + 1 : w);
        __syncthreads();                                           // shares in LDS; predictions and -Bm of the window before are read
        store_inputs(in, tab);
        hint.x2p = in.x2p;                                         // (not what the chain leaves, the Gram matrix's: launches end where they will)
        {
            const float *part = reinterpret_cast<const float *>(lds + Lds::part);
            double *q0d = reinterpret_cast<double *>(lds + Lds::q0);
#pragma unroll
            for (int u = 0; u < kB * kM / kRT; ++u) {
                const int e = tid + u * kRT;
                double sum = 0.0;
#pragma unroll
                for (int v = 0; v < kRW; ++v) sum += (double)part[v * kB * kM + e];
                q0d[(e >> 4) * kQStride + (e & 15)] = (e >> 4) < wl ? sum : 0.0;
            }
            if constexpr (DEEP) sum_gram_shares(wl);
        }
        __syncthreads();
        afresh();
        RowsU xu[2], xut;
        RowsQ xq[2], xqt;
        if (wave < 4) {
            if (q_lo + 4 * wave < q_hi) {                          // (wavefronts without a learner have no rounds)
                if (k > 0) n2 = measured_n2(4 * wave + lk);
                (void)chain_rounds<LOSS, Lds, OPT>(lds, 0, wave, lane, wl, eta, (double)a.D, scale, scale, n2, &hint, tab);
                scale = 1.0;
            }
        } else if (more) {
            gram(ahead, plan.len(w + 1), Lds::tables - tab);
        }
        // the rows of the first blocks (past the last block: rounds or zeros that are not used)
        static_for<2>([&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value;
            if (nth_block(b) < nfull) {
                rows.u(d, offu, nth_block(b), xu[b]);
                ahead.q(d, offq, nth_block(b), xq[b]);
            } else {
                none(xq[b], xu[b]);
            }
        });
        if (has_tail()) {
            rows.u(d, offu, nfull, xut);
            ahead.q(d, offq, nfull, xqt);
        } else {
            none(xqt, xut);
        }
        __syncthreads();
        afresh();
        load_inputs(more ? w + 1 : w, in);
        {
            const int ws = plan.start(w);
            const float *zb = reinterpret_cast<const float *>(lds + Lds::zb);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int l = wave + kRW * i, q = q_lo + l;
                if (q < q_hi && lane < wl)
                    a.Z[(int64_t)(q / K) * a.zl.zs_r + (int64_t)(q % K) * a.zl.zs_i + (int64_t)(ws + lane) * a.zl.zs_t] = zb[l * kYStride + lane];
            }
        }
        const float *bml = reinterpret_cast<const float *>(lds + Lds::bm) + lk * kBmStride + lr;
        float bmr[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) bmr[i] = bml[4 * i * kBmStride];
        const float F = reinterpret_cast<const float *>(lds + Lds::fv)[lr];
        f4 acc[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[rb] = f4{0.f, 0.f, 0.f, 0.f};
        float nn = 0.f;
        auto update = [&](const RowsU &x, const f4 &v) __attribute__((always_inline)) {
            f4 vb, vo = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r) vb[r] = v[r] * F;
#pragma unroll
            for (int i = 0; i < 16; i += 2) {
                vb = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[i], bmr[i], vb, 0, 0, 0);
                vo = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[i + 1], bmr[i + 1], vo, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) vb[r] += vo[r];
            return vb;
        };
        static_for<NB>([&](auto bc) __attribute__((always_inline)) {
            constexpr int b = decltype(bc)::value;
            const int blk = nth_block(b);
            if (blk < nfull) {
                V[b] = update(xu[b & 1], V[b]);
                if constexpr (b + 2 < NB) rows.u(d, offu, nth_block(b + 2), xu[b & 1]);
#pragma unroll
                for (int r = 0; r < 4; ++r) nn = fmaf(V[b][r], V[b][r], nn);
                q_of(xq[b & 1], V[b], acc);
                if constexpr (b + 2 < NB) ahead.q(d, offq, nth_block(b + 2), xq[b & 1]);
            }
        });
        if (has_tail()) {
            V[NB] = update(xut, V[NB]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                V[NB][r] = tail_in(r) ? V[NB][r] : 0.f;
                nn = fmaf(V[NB][r], V[NB][r], nn);
            }
            mask_q(xqt);
            q_of(xqt, V[NB], acc);
        }
        reinterpret_cast<float *>(lds + Lds::n2)[(wave * 4 + lk) * kM + lr] = nn;
        put_share(acc);
    }
    // ---- state out: the iterates themselves (scale 1) and their squared norms ----------------------
    afresh();
    const bool q_out = q_lo + lr < q_hi;
    float *vout = a.V + (int64_t)(q_out ? q_lo + lr : q_lo) * d + 4 * lk;
    static_for<NB>([&](auto bc) __attribute__((always_inline)) {
        constexpr int b = decltype(bc)::value;
        const int blk = nth_block(b);
        if (blk < nfull && q_out) *reinterpret_cast<f4u *>(vout + blk * 16) = V[b];
    });
#pragma unroll
    for (int r = 0; r < 4; ++r)
        if (has_tail() && q_out && tail_in(r)) vout[nfull * 16 + r] = V[NB][r];
    __syncthreads();
    if (wave < 4) {
        const double m2 = measured_n2(4 * wave + lk);
        const int q = q_lo + 4 * wave + lk;
        if (q < q_hi && lr == 0) {
            a.sigma[q] = 1.f;
            a.n2[q] = m2;
            if (OPT) { a.ha[q] = hint.ha; a.hp[q] = hint.hp; }
        }
    }
}

// The comparators' predictions <u_t[r], x_t> of streams of their own: a wavefront takes 16 rounds of a run, four at a time.
__global__ void __launch_bounds__(256) run_comparator_kernel(const DenseArgs a)
{
    const int lane = threadIdx.x & 63, r = (int)blockIdx.y, d = a.d;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int t_lo = ((int)blockIdx.x * 4 + wave) * 16, t_hi = min(t_lo + 16, a.n);
    if (t_lo >= a.n) return;
    int seg = 0;
    while (seg + 1 < a.S && a.seg_start[seg + 1] <= a.t0 + t_lo) ++seg;
    float *z = a.Z + (int64_t)r * a.zl.zs_r + (int64_t)a.K * a.zl.zs_i;
    for (int t = t_lo; t < t_hi;) {
        while (seg + 1 < a.S && a.seg_start[seg + 1] <= a.t0 + t) ++seg;
        int end = min(t + 4, t_hi);                                // ... of one segment
        if (seg + 1 < a.S && a.seg_start[seg + 1] < a.t0 + end) end = (int)(a.seg_start[seg + 1] - a.t0);
        const float *u = a.u + ((int64_t)r * a.S + seg) * d;
        const float *x = a.x + (int64_t)r * a.x_run_stride + (int64_t)t * d;
        const int64_t last = (int64_t)(end - 1 - t) * d;           // (rounds past the segment: its last one again)
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int j = lane; j < d; j += kWave) {
            const float uj = u[j];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] = fmaf(uj, x[min((int64_t)i * d, last) + j], acc[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int s = 32; s > 0; s >>= 1) acc[i] += __shfl_xor(acc[i], s);
            if (lane == 0 && t + i < end) z[(int64_t)(t + i) * a.zl.zs_t] = acc[i];
        }
        t = end;
    }
}

using RunKernel = void (*)(const DenseArgs, WinPlanD, int, int, int);
template <int LOSS, bool OPT> RunKernel pick_run_kernel(int nfull)
{
    if (nfull <= 2 * kRW) return dense_run_kernel<LOSS, OPT, 2>;
    if (nfull <= 4 * kRW) return dense_run_kernel<LOSS, OPT, 4>;
    if (nfull <= 8 * kRW) return dense_run_kernel<LOSS, OPT, 8>;
    return dense_run_kernel<LOSS, OPT, 16>;
}

}  // namespace

// Measured per pass, ms, register kernel / this one, plain squared loss, 3000 rounds: streams of their own, 1 run of 4 learners, 64 of 15,
// 256 of 5, 200 of 24:
//   d = 10    0.60 / 0.40   0.70 / 0.53   0.77 / 0.52   1.36 / 1.02        d = 777   1.70 / 1.19   1.90 / 1.42   2.14 / 2.23   5.13 / 3.46
//   d = 100   0.64 / 0.47   0.76 / 0.58   0.89 / 0.59   1.48 / 1.16        d = 1000  1.17 / 1.35   1.41 / 1.65       -         4.14 / 3.72
//   d = 256   0.71 / 0.64   0.87 / 0.69   0.99 / 0.88   2.16 / 1.45        d = 2048  1.73 / 2.32   2.24 / 2.88       -           -
//   d = 500   0.86 / 0.84   1.04 / 0.98   1.27 / 1.34   2.76 / 2.16        (1000 rounds, 200 of 24: d = 1500 2.64 / 2.06, d = 2048 2.83 / 2.33)
// so the line lies at d = 448 where rows are aligned, at 1024 where they are not (the register kernel copies those word by word; 16 runs
// of 8, d = 777 1.73 / 1.23), and at the last d the kernel holds where the register kernel has four wavefronts and more on every SIMD.
// A shared stream, 1 / 256 / 2048 learners: d = 10 0.60 / 0.39, 0.64 / 0.45, 0.81 / 0.55; d = 400 0.85 / 0.76, 0.88 / 0.80, 1.05 / 0.85; d = 512 0.85 /
// 0.84, 0.88 / 0.89, 1.11 / 0.94; d = 501, 256 learners 1.13 / 0.88.  More learners than dense_split.hip takes stay where they are.  Of 600
// rounds the two took the same when these calls too went in four pieces (d = 100 0.223 / 0.222 and 0.203 / 0.205), 1000 of one learner 0.250 /
// 0.198, now 0.179: hence the least n.  The horizon's
// last call, which is as short as the cuts leave it, stays with the kernel of the calls before it, as in dense_split.hip.
// (The rules look at the configuration and the call's length only, not at addresses.)
//
// A workgroup takes a compute unit's LDS, so more than 256 of them are turns of the chip, each as long whether its tiles hold one
// learner or sixteen, while what the register kernel takes goes by its wavefronts.  Streams of their own, 1200 rounds, the same loss, ms, learners x runs:
//               1 x 1024      4 x 1024      8 x 512       17 x 256      16 x 258      16 x 1024     32 x 512
//   d = 64      0.53 / 0.70   0.63 / 0.72   0.50 / 0.44   0.51 / 0.46   0.58 / 0.50   1.72 / 0.96   1.73 / 0.98
//   d = 448     1.33 / 1.85   1.26 / 1.85   0.84 / 1.01   0.78 / 0.89   1.07 / 0.89   2.74 / 2.05   2.72 / 1.90
//   d = 1000    1.87 / 3.57   2.07 / 3.66   1.31 / 1.98   1.12 / 1.70   1.35 / 1.56   4.98 / 3.87   3.87 / 3.50
// So beyond a turn tiles have to be three quarters full, half where the sweeps are short beside the rounds (512 runs of 8: d = 192 0.64 / 0.60, but
// 448 as above; longer rows that the register kernel copies word by word), all of wide aligned models; and of
// aligned models the register kernel needs 2, 2.75 or 3 wavefronts per SIMD and turn as they get wider (d = 1000, 300 runs of sixteen,
// 2.5 of them 1.46 / 1.66; 640 runs, 3.5 of them 3.27 / 2.77).  Within a turn workgroups slow each other only by their draw on the caches: from 161 of
// them and d = 321 tiles have to be half full, beyond d = 800 from 129 (800 rounds of d = 448, 192 runs of one learner 0.34 / 0.39, of sixteen
// 0.50 / 0.43; optimistic, d = 1001, 160 runs of one 0.65 / 0.74).  A run of
// up to fifteen learners and its comparator is one workgroup of the register kernel, which a compute unit works as fast as a wavefront or two
// per SIMD: such runs of wide aligned models stay there (256 of fifteen, d = 2048 1.70 / 1.91; of sixteen 2.54 / 1.92).
bool dense_run_wanted(const DenseArgs &a)
{
    if (a.tune->get(OCO_OPT_DENSE_PATH) >= 0 || a.tune->get(OCO_OPT_WINDOW_RESIDENT) >= 0 || a.tune->get(OCO_OPT_DENSE_HALF) >= 0 ||
        a.tune->get(OCO_OPT_COMPARATOR_GEMM) == 0)
        return false;                                               // (a choice that only the register kernel has, of those that may regroup sums)
    if (!a.scaled) return false;
    constexpr int kSimds = 1024;
    const int64_t waves = (int64_t)a.R * (a.K + 1);                 // of the register kernel
    const bool aligned = a.d % 4 == 0;
    int most = aligned ? 448 : 1024;
    if (a.x_shared) {
        if ((int64_t)a.R * a.K > 2048) return false;
    } else {
        constexpr int kUnits = 256;
        const int64_t tiles = (a.K + kM - 1) / kM, wgs = a.R * tiles, turns = (wgs + kUnits - 1) / kUnits;
        const bool narrow = a.d <= (aligned ? 192 : 320), full = aligned && a.d > 800;
        if (turns > 1) {
            const int64_t quarters = narrow || !aligned ? 0 : full ? 12 : a.d > 448 ? 11 : 8;    // of a wavefront per SIMD
            if (a.K < (narrow ? 8 : full ? 16 : 12) * tiles || waves * 4 < quarters * kSimds * turns) return false;
        } else if (wgs > (a.d > 800 ? 128 : 160) && a.d > 320 && a.K < 8 * tiles) {
            return false;
        }
        if (waves >= 4 * kSimds) most = aligned && a.K < 16 ? 800 : 16 * kRunMaxBlocks;
        else if (waves >= kSimds && !aligned) most = 640;
    }
    const bool rest = a.plan->after_split && a.t0 + a.n == a.T;
    return a.d <= most && (a.n >= 768 || rest);
}

hipError_t launch_dense_run(const DenseArgs &a, int loss, hipStream_t s, const PieceHook *hook)
{
    if (a.n <= 0) return hipSuccess;
    const WinPlanD plan{a.t0, a.n};
    const int nwin = plan.count(), nfull = a.d / 16;
    RunKernel kern = nullptr;
    switch (loss * 2 + (a.optimistic ? 1 : 0)) {
        case 0: kern = pick_run_kernel<0, false>(nfull); break;
        case 1: kern = pick_run_kernel<0, true>(nfull); break;
        case 2: kern = pick_run_kernel<1, false>(nfull); break;
        case 3: kern = pick_run_kernel<1, true>(nfull); break;
        case 4: kern = pick_run_kernel<2, false>(nfull); break;
        case 5: kern = pick_run_kernel<2, true>(nfull); break;
        default: return hipErrorInvalidValue;
    }
    const int lds_bytes = nfull <= 2 * kRW ? LdsR<false>::total : LdsR<true>::total;
    // tiles: of a run (its learners dealt evenly), or of all learners of a shared stream
    const int learners = a.x_shared ? a.R * a.K : a.K;
    const int tiles = (learners + kM - 1) / kM, per_tile = a.x_shared ? kM : (learners + tiles - 1) / tiles;
    const int64_t wgs = (int64_t)tiles * (a.x_shared ? 1 : a.R);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    if (a.tune->get(OCO_OPT_VERBOSE) == 1)
        fprintf(stderr, "dense plan: windows of a stream's own Gram matrices, %d windows, %lld workgroups of %d learners\n", nwin, (long long)wgs, per_tile);
    if (a.optimistic) {
        e = launch_hint_scalars(a, s);
        if (e != hipSuccess) return e;
    }
    // The caller's work on a piece's rounds (the meta kernel) goes beside the following piece where compute units are left, and where a call is
    // long enough for that to be worth the events and launches it takes (ms beside / behind, learners of one stream: 800 rounds, 1 of d = 10
    // 0.189 / 0.162, 8 of d = 448 0.325 / 0.297, the register kernel 0.309; 1100 rounds 0.211 / 0.196 and 0.399 / 0.384; 1600 rounds 0.253 / 0.255
    // and 0.508 / 0.510), or the comparators' contraction over a shared stream is: 960 of d = 777, 800 rounds 0.459 / 0.493.
    const bool worth = a.n >= 1152 || (a.x_shared && a.d > 448);
    const bool beside = hook && hook->fn && hook->beside && wgs <= 192 && worth;
    hipStream_t cs = s;
    if (beside) e = hook->beside(hook->ctx, &cs);                   // only the meta kernel reads the comparators' predictions
    if (e != hipSuccess) return e;
    if (a.x_shared) {
        ComparatorGemmArgs g{};
        g.x = a.x; g.u = a.u; g.seg_start = a.seg_start; g.S = a.S; g.Z = a.Z; g.zl = a.zl;
        g.d = a.d; g.K = a.K; g.R = a.R; g.t0 = a.t0; g.n = a.n; g.vec_ok = a.vec_ok;
        e = launch_comparator_gemm(g, cs);
    } else {
        hipLaunchKernelGGL(run_comparator_kernel, dim3((unsigned)((a.n + 63) / 64), (unsigned)a.R), dim3(256), 0, cs, a);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    // pieces of 4, 3, 2 and 1 tenths of the windows: what follows the last is the meta work of a tenth (as many equal ones as the option
    // asks for, none shorter than the register kernel's)
    const int64_t asked = std::min<int64_t>(a.tune->get(OCO_OPT_DENSE_PIECES), std::max(a.n / 512, 1));
    const int pieces = asked >= 1 ? (int)asked : beside ? 4 : 1;
    auto piece_end = [&](int i) { return asked >= 1 ? (int)((int64_t)nwin * (i + 1) / pieces) : nwin * (i == 0 ? 4 : i == 1 ? 7 : 9) / 10; };
    int done = 0, w0 = 0;
    for (int i = 0; i < pieces && w0 < nwin; ++i) {
        const int w1 = i == pieces - 1 ? nwin : std::min(nwin, std::max(w0 + 1, piece_end(i)));
        e = clock_begin(a.clock, s, "dense_window_kernel");
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)(a.x_shared ? 1 : a.R)), dim3(kRT), lds_bytes, s, a, plan, w0, w1 - w0, per_tile);
        e = hipGetLastError();
        if (e == hipSuccess) e = clock_end(a.clock, s);
        const int end = plan.start(w1 - 1) + plan.len(w1 - 1);
        if (e == hipSuccess && beside) e = hook->fn(hook->ctx, done, end - done);
        if (e != hipSuccess) return e;
        done = end;
        w0 = w1;
    }
    return a.optimistic ? launch_keep_last_row(a, s) : hipSuccess;
}

}  // namespace oco
