// Dense rounds of the base learners on a shared round stream, worked in windows of 64 rounds as
// contractions on the matrix cores (Sec. 3.1 update inside the ensemble of Sec. 3.3).
//
// The update of a base learner, w_{t+1} = Proj[w_t - eta c_t x_t] with c_t = phi'(<w_t, x_t>; y_t),
// keeps the iterate in the span of the window's start w_s and the window's round rows, whatever
// the projections do (a projection onto the ball only rescales):
//     w_t = A_t w_s - sum_{s <= r < t} a_r rho_{r,t} x_r,   a_r = eta c_r,
//     rho_{r,t} = f_r f_{r+1} ... f_{t-1},   A_t = f_s ... f_{t-1},   f_r = min(1, D / ||w_r - a_r x_r||).
// So for a window of B = 64 rounds and a tile of M = 16 learners (any 16 learners: the stream is
// shared), with W the M x d matrix of iterates and X_w the B x d block of round rows:
//   (1) Q0 = W X_w^T                                  (M x B contraction over d, matrix cores)
//   (2) the 64 dependent rounds on scalars only: with G = X_w X_w^T (once per window for all
//       learners, pre-pass), p_{t2} = <w_t, x_{t2}> for the rounds t2 >= t still to come obeys
//           p_{t2} <- f_t (p_{t2} - a_t G[t][t2]),
//       the prediction of round t is p_t itself, and the squared norm follows from
//           ||w_t - a_t x_t||^2 = ||w_t||^2 - 2 a_t <w_t, x_t> + a_t^2 G[t][t]
//       (float64 scalars; one wavefront, a quad of lanes per learner, each lane of the quad
//       carrying every fourth pending round);
//   (3) W <- F W - Bm X_w,  F = A_end,  Bm[r] = a_r rho_{r,end}   (M x d contraction over B).
// The dependent rounds (2) occupy one wavefront; so that the matrix cores do not wait for them,
// (2) of window k runs beside the sweep that applies (3) of window k - 1.  Its inner products
// cannot then be taken with w_k itself (not formed yet); the sweep before took Q' = W_{k-1} X_k^T,
// and with W_k = F W_{k-1} - Bm X_{k-1},
//     Q0_k = F Q' - Bm (X_{k-1} X_k^T),
// a 16 x 64 x 64 contraction with the cross Gram matrix of the two windows (pre-pass), four
// matrix instructions deep.  One sweep over the coordinates per window, block by block:
// (3) of window k - 1, then that block's share of W_k X_{k+1}^T, so the iterates are touched once
// per window.  ||w||^2 is carried through the windows by the scalar identity above (float64) and
// re-anchored one window late on the exact sum of squares that the sweep takes of the new iterates.
//
// The iterates live in HBM between windows: the sweep loads each 16 x 16 block, updates it, takes
// its share of the next window's inner products and writes it back, 8 bytes per coordinate,
// learner and window, all in full 64-byte segments.  A workgroup works two tiles, so that every
// round row a wavefront loads (from L2: all tiles read the same rows) serves 32 learners; a
// compute unit draws only about 21 bytes per clock from L2, which is what bounds the sweep.
// Variants (OCO_OPT_WINDOW_RESIDENT): the iterates of one tile held in the registers of the
// workgroup for a whole launch (d <= 4096: eight wavefronts, each with every eighth block, in
// the layout the matrix instruction writes: a lane holds 4 coordinates of one learner); those of
// two tiles (d <= 1024; the default for 512 <= d <= 1024: a window's time is then the dependent
// rounds plus the sweep of the wavefronts that ran them, and without the iterates' loads and stores
// the sweep is bound by the matrix instructions of each SIMD); and one streamed tile worked by
// sixteen wavefronts.
//
// v_mfma_f32_16x16x4_f32 computes D = A B + C with A 16x4, B 4x16: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and holds D[4 (l / 16) + r][l % 16] in register r.
// A block of iterates is kept as the transposed 16 coordinates x 16 learners D tile, so that
// register r of it is at once the B operand of (1) for the depth indices k <-> coordinate 4 k + r
// (the order of the terms of an inner product is free; the round rows are laid out to match).
//
// The round rows as operands.  In (1) a lane holds (round l % 16, four coordinates): read from
// the stream, neighbouring lanes would sit in different rows, 16 bytes each.  A pre-pass
// therefore re-tiles the stream once per launch: per window and block of 16 coordinates, 4 KB in
// the order the lanes of (1) want them and 4 KB in the order the lanes of (3) want them (lane:
// coordinate l % 16, sixteen rounds), so that every load of the sweep is 16 bytes per lane and
// 1 KB contiguous per instruction, rows past a window's length and coordinates past d already
// zero.  A call is worked in pieces of at most 64 MB of stream so that the two copies stay a
// bounded scratch (and, with the piece itself, inside the last-level cache for every tile).
//
// Windows end at the multiples of 64 of the horizon; a call that starts or ends elsewhere has
// shorter first / last windows.
#include "dense_window_common.h"
#include "../../include/oco.h"

#include <algorithm>
#include <cstdio>

namespace oco {
namespace {

constexpr int kNW8 = 8;           // wavefronts per workgroup: iterates in registers (two per SIMD, 256 registers each)
constexpr int kNW16 = 16;         // ... iterates streamed from HBM (four per SIMD: a wavefront's loads hide behind the others' work)

// (A build with -DOCO_WIN_PROF keeps wall-clock sums of the phases of workgroup 0's window loop in g_win_prof,
// read back through oco_debug_win_prof: how the figures per phase in the comments below were taken.)
#ifdef OCO_WIN_PROF
__device__ unsigned long long g_win_prof[8];
#ifndef OCO_WIN_PROF_TID
#define OCO_WIN_PROF_TID 0
#endif
#define PROF_T(i) do { if (threadIdx.x == OCO_WIN_PROF_TID) { const unsigned long long now_ = wall_clock64(); prof_[i] += now_ - last_; last_ = now_; } } while (0)
#else
#define PROF_T(i) do { } while (0)
#endif

// ---- pre-pass 1: the round rows of the windows w0 .. w0 + gridDim.y - 1, re-tiled ----------------
// One wavefront per (window, block of 16 coordinates).  xq[((w - w0) nblk + blk) 1024 + (rb 64 + l) 4 + r]
// = x[round 16 rb + l % 16][coordinate 16 blk + 4 (l / 16) + r], xu[... + (k 64 + l) 4 + r]
// = x[round 4 (4 k + r) + l / 16][coordinate 16 blk + l % 16]; zero past the window or past d.
__global__ void __launch_bounds__(64) dense_tile_kernel(const float *x, int d, WinPlanD plan, int w0, float *xq, float *xu,
                                                        float *misc)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kMiscZeros) misc[threadIdx.x] = 0.f;   // see kMiscZeros
    const int blk = blockIdx.x, w = w0 + blockIdx.y;
    const int nblk = gridDim.x;
    const int ws = plan.start(w), wl = plan.len(w);
    const int l = threadIdx.x, lr = l & 15, lk = l >> 4;
    const int64_t tile = ((int64_t)blockIdx.y * nblk + blk) * kTileFloats;
    const float *xw = x + (int64_t)ws * d + blk * 16;
    {
        const int c = blk * 16 + 4 * lk;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const int t = rb * 16 + lr;
            f4 v = f4{0.f, 0.f, 0.f, 0.f};
            if (c < d && t < wl) v = *reinterpret_cast<const f4 *>(xw + (int64_t)t * d + 4 * lk);
            *reinterpret_cast<f4 *>(xq + tile + (rb * 64 + l) * 4) = v;
        }
    }
    if (xu) {
        const int c = blk * 16 + lr;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = 4 * (4 * k + r) + lk;
                v[r] = (c < d && t < wl) ? xw[(int64_t)t * d + lr] : 0.f;
            }
            *reinterpret_cast<f4 *>(xu + tile + (k * 64 + l) * 4) = v;
        }
    }
}

// ---- rows and iterates as three bfloat16 parts ---------------------------------------------------
// (The splitting of Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision
// computations", ARITH 2019.)  v = v1 + v2 + v3, each part the bfloat16 nearest to what the ones before leave: 3 x 8 bits hold all 24 of a
// float32.  A product of two such numbers is taken as its six largest part products, each exact in float32, by the
// 16-bit matrix instructions: dropped are (2,3), (3,2) and (3,3), at most 2^-24 of the product (|v2| <= 2^-8 |v|, |v3| <= 2^-17 |v|), 2^-27.5 in the mean square;
// six products cost 0.375 of the time of the float32 instructions' one.
typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
constexpr int kSplitFloats = kTileFloats * 3 / 2;            // one window x one block, split: 6 KB

// two neighbouring values: their first, second and third parts, packed
__device__ __forceinline__ void split2(float a, float b, unsigned &p1, unsigned &p2, unsigned &p3)
{
    auto pack = [](float x, float y) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f2{x, y}, bf2)); };
    auto lo = [](unsigned p) { return __uint_as_float(p << 16); };
    auto hi = [](unsigned p) { return __uint_as_float(p & 0xFFFF0000u); };
    p1 = pack(a, b);
    const float ra = a - lo(p1), rb = b - hi(p1);
    p2 = pack(ra, rb);
    p3 = pack(ra - lo(p2), rb - hi(p2));
}
__device__ __forceinline__ f4 mfma_bf16(u4 a, u4 b, f4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// The round rows of the windows w0 .. w0 + gridDim.y - 1 in parts, as dense_window_shared_kernel wants them.  v_mfma_f32_16x16x32_bf16
// takes A 16x32 and B 32x16, lane l with A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16]; which depth index is which
// coordinate or round is free.  One wavefront per (window, block of 16 coordinates), 16 bytes per lane and KB:
//   xq: KB rb = 0 .. 3: parts 1 (four coordinates 4 (l / 16) ..) and 2 of round 16 rb + l % 16; KB 4, 5: part 3 of rounds
//       16 rb + l % 16 for rb = 0, 1 and 2, 3 -- a depth of 32 is the block's 16 coordinates for two products at once;
//   xu: KB 2 p + s: part p of coordinate l % 16, rounds 32 s + 8 (l / 16) ..
__global__ void __launch_bounds__(64) dense_tile_split_kernel(const float *x, int d, WinPlanD plan, int w0, float *xq, float *xu)
{
    const int blk = blockIdx.x, w = w0 + blockIdx.y, nblk = gridDim.x;
    const int ws = plan.start(w), wl = plan.len(w);
    const int l = threadIdx.x, lr = l & 15, lk = l >> 4;
    const int64_t tile = ((int64_t)blockIdx.y * nblk + blk) * kSplitFloats;
    const float *xw = x + (int64_t)ws * d + blk * 16;
    {
        u4 *out = reinterpret_cast<u4 *>(xq + tile) + l;
        u4 third[2];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            const int t = rb * 16 + lr;
            f4 v = f4{0.f, 0.f, 0.f, 0.f};
            if (blk * 16 + 4 * lk < d && t < wl) v = *reinterpret_cast<const f4 *>(xw + (int64_t)t * d + 4 * lk);
            unsigned a1, a2, a3, b1, b2, b3;
            split2(v[0], v[1], a1, a2, a3);
            split2(v[2], v[3], b1, b2, b3);
            out[rb * 64] = u4{a1, b1, a2, b2};
            third[rb >> 1][2 * (rb & 1)] = a3;
            third[rb >> 1][2 * (rb & 1) + 1] = b3;
        }
        out[4 * 64] = third[0];
        out[5 * 64] = third[1];
    }
    {
        u4 *out = reinterpret_cast<u4 *>(xu + tile) + l;
        const int c = blk * 16 + lr;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            u4 p[3];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = 32 * s + 8 * lk + 2 * j;
                const float v0 = (c < d && t < wl) ? xw[(int64_t)t * d + lr] : 0.f;
                const float v1 = (c < d && t + 1 < wl) ? xw[(int64_t)(t + 1) * d + lr] : 0.f;
                unsigned q1, q2, q3;
                split2(v0, v1, q1, q2, q3);
                p[0][j] = q1; p[1][j] = q2; p[2][j] = q3;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) out[(2 * k + s) * 64] = p[k];
        }
    }
}

// ---- pre-pass 2: G = X_w X_w^T of the same windows, from the tiled rows, and the cross Gram
// matrix Gx[r][t] = <x_r of window w - 1, x_t of window w> for every window but the launch's first.
// One workgroup of eight wavefronts per window; wavefronts 0..3 compute rows 16 v .. 16 v + 15 of G
// (four 16 x 16 blocks), wavefronts 4..7 the same rows of Gx, depth block by block.  Fixed
// summation order.  Gx is written in the order the round kernel's matrix instructions want it:
// gxt[((t / 16) 4 + r / 16) 256 + (t % 16 + 16 (r % 4)) 4 + (r / 4) % 4].
__global__ void __launch_bounds__(512) dense_gram_kernel(const float *xq, int nblk, float *gram, float *gxt)
{
    const int lane = threadIdx.x & 63, wave8 = threadIdx.x >> 6;
    const int wave = wave8 & 3;
    const bool cross = wave8 >= 4;
    if (cross && blockIdx.x == 0) return;
    const int lr = lane & 15, lk = lane >> 4;
    f4 acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = f4{0.f, 0.f, 0.f, 0.f};
    const float *xw = xq + (int64_t)blockIdx.x * nblk * kTileFloats + lane * 4;          // this window
    const float *xa = cross ? xw - (int64_t)nblk * kTileFloats : xw;                     // rows: the window before, or this one
    for (int blk = 0; blk < nblk; ++blk) {
        f4 bv[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) bv[b] = *reinterpret_cast<const f4 *>(xw + (int64_t)blk * kTileFloats + b * 256);
        const f4 av = *reinterpret_cast<const f4 *>(xa + (int64_t)blk * kTileFloats + wave * 256);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[r], bv[b][r], acc[b], 0, 0, 0);
    }
    // acc[b][r]: row 16 wave + 4 lk + r, column 16 b + lr
    if (!cross) {
        float *g = gram + (int64_t)blockIdx.x * kB * kB;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[(wave * 16 + 4 * lk + r) * kB + b * 16 + lr] = acc[b][r];
    } else {
        float *g = gxt + (int64_t)blockIdx.x * kB * kB;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) g[(b * 4 + wave) * 256 + (lr + 16 * r) * 4 + lk] = acc[b][r];
    }
}

// LDS of the window kernel (dynamic), in bytes from the base.  What the dependent rounds of window
// k write for the sweep (predictions, -Bm, F) and the labels staged for them have two buffers,
// window k in buffer k % 2: the sweep of window k - 1 and the staging for window k + 1 run beside
// them.  The Gram table (float64, its diagonal in the rows' padding) has one: it is written
// between the two barriers that precede the rounds, from registers loaded before the first.
// MT: tiles of 16 learners per workgroup (per-tile arrays come MT times; the Gram table and the
// shares' buffer are common).
template <int NW, int MT> struct LdsT {
    // float64 where the LDS has room (one tile, eight wavefronts), else float32
    static constexpr bool wide = NW == kNW8 && MT == 1;
    using G = double;                                              // Gram table
    using S = std::conditional_t<wide, double, float>;             // inner products handed to the rounds, f_t
    static constexpr int g_reads = 1;                               // how the rounds read the Gram table (chain_window)
    static constexpr bool carry_norm = false;
    static constexpr bool has_corr = true;                         // the rounds start from pmul q0 + corr
    static constexpr int gd_bytes = kB * 4 * kGStride * (int)sizeof(G);   // G [64][4][kGStride]: G[t][t2], zero for t2 <= t;
                                                                   //   [t][0][16] holds G[t][t]
    static constexpr int tile_f = kB * kM * 4;                     // float [64][16]
    static constexpr int tile_s = kB * kM * (int)sizeof(S);        // S [64][16]
    static constexpr int yb_bytes = MT * tile_f;                   // labels
    static constexpr int zb_bytes = MT * tile_f;                   // predictions
    static constexpr int bm_bytes = MT * tile_f;                   // -Bm
    static constexpr int fv_bytes = MT * kM * 4;                   // float [16]: F
    static constexpr int gd = 0;
    static constexpr int yb = gd + gd_bytes;
    static constexpr int zb = yb + 2 * yb_bytes;
    static constexpr int bm = zb + 2 * zb_bytes;
    static constexpr int fv = bm + 2 * bm_bytes;
    static constexpr int q0 = fv + 2 * fv_bytes;                   // S [MT][64][16]: W' X_k^T
    static constexpr int fl = q0 + MT * tile_s;                    // S [MT][64][16]: f_t
    static constexpr int part = fl + MT * tile_s;                  // float [NW][64][16]: per-wavefront shares of W X^T (one tile at a time)
    static constexpr int st = part + NW * tile_f;                  // float [MT][64][16]: a_t
    static constexpr int corr = st + MT * tile_f;                  // float [MT][64][16]: -Bm (X_{k-1} X_k^T)
    static constexpr int n2 = corr + MT * tile_f;                  // float [MT][NW][4][16]: shares of ||w||^2
    static constexpr int hg = n2 + MT * NW * 4 * kM * 4;           // float [2][64]: <x_{t-1}, x_t> of the window's rounds (optimistic update)
    static constexpr int hg_bytes = kB * 4;
    static constexpr int total = hg + 2 * hg_bytes;
};
static_assert(LdsT<kNW8, 1>::total <= 160 * 1024 && LdsT<kNW16, 1>::total <= 160 * 1024 && LdsT<kNW8, 2>::total <= 160 * 1024,
              "LDS of a gfx950 compute unit");

// What a thread is in the sweep, derived from its index.  The window loop re-derives it every
// iteration from an index the compiler cannot see through, so that none of it (nor the many
// addresses that follow from it) is kept alive across the dependent rounds.
template <int MT> struct Geo {
    int tid, lane, wave, lr, lk;
    bool q_ok[MT];             // this lane's learner of tile m exists
    float *vrow[MT];           // its row of the iterates, at this lane's 4 coordinates of a block
};
template <int MT> __device__ __forceinline__ Geo<MT> make_geo(int tid, const DenseArgs &a)
{
    Geo<MT> g;
    g.tid = tid;
    g.lane = tid & 63;
    g.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    g.lr = g.lane & 15;
    g.lk = g.lane >> 4;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int q = ((int)blockIdx.x * MT + m) * kM + g.lr;
        g.q_ok[m] = q < a.R * a.K;
        g.vrow[m] = a.V + (int64_t)(g.q_ok[m] ? q : 0) * a.d + 4 * g.lk;
    }
    return g;
}

// The windows w0 .. w0 + nw - 1 of the call's plan; xq / xu / gram / gxt hold those windows only.
// RES: the iterates stay in registers for the whole launch (one tile, d <= 16 * NW * NB); otherwise
// every block is loaded and stored in the sweep.  NW: wavefronts per workgroup.  MT: tiles of 16
// learners per workgroup -- with two, a wavefront uses every round row it loads for both (a compute
// unit draws only about 21 bytes per clock from L2, and the sweep of one tile needs 8 KB of rows per
// 32 matrix instructions); wavefront m runs the dependent rounds of tile m.
//
// Iteration k = 0 .. nw of the main loop:
//   all        the shares of W' X_k^T -> q0, tile by tile; four wavefronts per tile: corr = -Bm_{k-1} Gx_k (k >= 1)
//   wavefronts < MT    the dependent rounds of window k (k < nw), then their part of the sweep
//   the others     predictions of window k - 1 to Z, staging for window k + 1, the sweep
//   sweep (k >= 1) W_k = F_{k-1} W_{k-1} - Bm_{k-1} X_{k-1} block by block, its squared norm, and the
//                  shares of W_k X_{k+1}^T (k + 1 < nw)
template <int LOSS, int NB, bool RES, int NW, int MT, bool OPT = false>
__global__ void __launch_bounds__(NW *kWave) dense_window_kernel(const DenseArgs a, const float *gram, const float *gxt,
                                                                  const float *xq, const float *xu, float *misc,
                                                                  WinPlanD plan, int w0, int nw)
{
    static_assert(!RES || MT == 1 || (MT == 2 && NW == 8 && NB == 9), "iterates in registers: one tile, or two on eight wavefronts");
    using Lds = LdsT<NW, MT>;
    using GT = typename Lds::G;
    using ST = typename Lds::S;
    // -Bm in registers for the whole sweep, or (where registers are short) re-read from LDS per block
    constexpr bool BMR = RES && NB <= 8 && MT == 1;
    extern __shared__ __align__(16) char lds[];
    const int d = a.d, K = a.K;
    const int nq = a.R * K;
    const int nblk = (d + 15) / 16;                             // blocks of 16 coordinates
    const int q_base = (int)blockIdx.x * MT * kM;               // first learner of the workgroup

    // Which blocks of 16 coordinates a wavefront takes.  In registers: wave, wave + NW, ...  Streamed
    // with sixteen wavefronts: wavefront 0 also runs the dependent rounds, so it takes half a share:
    // of every 31 consecutive blocks, wavefronts 1 .. 15 take two each and wavefront 0 the last one.
    // (A fixed assignment: every sum keeps its order from run to run.)
    auto nth_block = [&](int wave, int i) __attribute__((always_inline)) {
        if (NW == kNW16 && !RES) {
            if (wave == 0) return 31 * i + 30;
            return 31 * (i >> 1) + (wave - 1) + ((i & 1) ? 15 : 0);
        }
        if (MT == 2) {
            // two tiles, eight wavefronts: wavefronts 0 and 1 run the dependent rounds first and take two
            // blocks of every 22, the other six three each
            if (wave < 2) return 22 * (i >> 1) + 6 + wave + 8 * (i & 1);
            return 22 * (i / 3) + (wave - 2) + 8 * (i % 3);
        }
        return wave + NW * i;
    };
    // Which wavefront runs the dependent rounds of which tile (-1: of none), and the number of a wavefront
    // among those that run none.  Two tiles in registers: wavefronts 0 and 4, which share a SIMD (a workgroup's
    // wavefronts are dealt to the four SIMDs in turn), so that the rounds do not share theirs with a wavefront
    // of matrix instructions (beside one they take 16 us per window instead of 10) and the other three SIMDs
    // have two sweeping wavefronts each.
    constexpr bool PAIR = RES && MT == 2;
    auto rounds_tile = [&](int wave) __attribute__((always_inline)) {
        if (PAIR) return (wave & 3) == 0 ? wave >> 2 : -1;
        return wave < MT ? wave : -1;
    };
    auto other_index = [&](int wave) __attribute__((always_inline)) {
        if (PAIR) return wave < 4 ? wave - 1 : wave - 2;
        return wave - MT;
    };
    // Iterates in registers: the b-th block a wavefront keeps.  One tile: wave, wave + NW, ...  Two tiles
    // (eight wavefronts, NB = 9, at most 64 blocks): the six wavefronts without dependent rounds keep blocks
    // 0 .. 53, nine each; the two with them sweep only when their rounds are done and keep blocks 54 .. 63:
    // wavefront 0, whose rounds the SIMD works first, seven of them, wavefront 4 three.
    auto kept_block = [&](int wave, int b) __attribute__((always_inline)) {
        if (PAIR) {
            if ((wave & 3) != 0) return other_index(wave) + 6 * b;
            return wave == 0 ? (b < 7 ? 54 + b : (1 << 20)) : (b < 3 ? 61 + b : (1 << 20));
        }
        return wave + NW * b;
    };
    // a tile's iterates: 16 coordinates x 16 learners per block, transposed
    auto ld_block = [&](const Geo<MT> &g, int m, int blk) __attribute__((always_inline)) {
        f4 v = f4{0.f, 0.f, 0.f, 0.f};
        if (g.q_ok[m] && blk * 16 + 4 * g.lk < d) v = *reinterpret_cast<const f4 *>(g.vrow[m] + blk * 16);
        return v;
    };
    auto st_block = [&](const Geo<MT> &g, int m, int blk, const f4 &v) __attribute__((always_inline)) {
        if (g.q_ok[m] && blk * 16 + 4 * g.lk < d) *reinterpret_cast<f4 *>(g.vrow[m] + blk * 16) = v;
    };
    // the same without a branch (streamed sweep): every lane loads and stores, the lanes without a
    // learner or past d from / to the scratch words
    auto ld_block_nb = [&](const Geo<MT> &g, int m, int blk) __attribute__((always_inline)) {
        const bool ok = g.q_ok[m] && blk * 16 + 4 * g.lk < d;
        const float *src = ok ? g.vrow[m] + blk * 16 : misc;
        return *reinterpret_cast<const f4 *>(src);
    };
    auto st_block_nb = [&](const Geo<MT> &g, int m, int blk, const f4 &v) __attribute__((always_inline)) {
        const bool ok = g.q_ok[m] && blk * 16 + 4 * g.lk < d;
        float *dst = ok ? g.vrow[m] + blk * 16 : misc + kMiscZeros + g.tid * 4;
        *reinterpret_cast<f4 *>(dst) = v;
    };
    // the tiled round rows of window wi (relative to w0), block blk: four 16-byte loads per lane each
    auto ldq = [&](const Geo<MT> &g, int wi, int blk, f4 (&o)[4]) __attribute__((always_inline)) {
        const float *t = xq + ((int64_t)wi * nblk + blk) * kTileFloats + g.lane * 4;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) o[rb] = *reinterpret_cast<const f4 *>(t + rb * 256);
    };
    auto ldu = [&](const Geo<MT> &g, int wi, int blk, f4 (&o)[4]) __attribute__((always_inline)) {
        const float *t = xu + ((int64_t)wi * nblk + blk) * kTileFloats + g.lane * 4;
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k] = *reinterpret_cast<const f4 *>(t + k * 256);
    };
    // The Gram matrix of window wi on its way to LDS: every thread carries kGPer consecutive entries
    // of a row in registers (loaded before a barrier, stored after it), masked to t2 > t, the
    // diagonal in the rows' padding.
    constexpr int kGPer = kB * kB / (NW * kWave);               // 8 or 4
    auto load_gram = [&](int tid, int wi, f4 (&gv)[kGPer / 4]) __attribute__((always_inline)) {
        const float *gsrc = gram + (int64_t)wi * kB * kB + tid * kGPer;
#pragma unroll
        for (int i = 0; i < kGPer / 4; ++i) gv[i] = *reinterpret_cast<const f4 *>(gsrc + 4 * i);
    };
    auto store_gram = [&](int tid, const f4 (&gv)[kGPer / 4]) __attribute__((always_inline)) {
        GT *gd = reinterpret_cast<GT *>(lds + Lds::gd);
        const int t = (tid * kGPer) >> 6, t2b = (tid * kGPer) & 63;
#pragma unroll
        for (int i = 0; i < kGPer; ++i) {
            const int t2 = t2b + i;
            const float v = gv[i >> 2][i & 3];
            gd[(t * 4 + (i & 3)) * kGStride + (t2 >> 2)] = t2 > t ? (GT)v : (GT)0;   // (t2b is a multiple of 4: t2 & 3 == i & 3)
            if (t2 == t) *reinterpret_cast<float *>(gd + t * 4 * kGStride + 16) = v;
        }
    };
    // LDS inputs of the dependent rounds of window wi: the labels.  `nthr` threads numbered tid share the work.
    auto stage_chain_inputs = [&](int tid, int nthr, int wi) __attribute__((always_inline)) {
        const int w = w0 + wi, buf = wi & 1;
        const int ws = plan.start(w), wl = plan.len(w);
        float *yb = reinterpret_cast<float *>(lds + Lds::yb + buf * Lds::yb_bytes);
        for (int e = tid; e < MT * kB * kM; e += nthr) {
            const int l = e >> 6, t = e & 63;                   // a learner's 64 labels are contiguous
            const int q = q_base + l;
            float yv = 0.f;
            if (a.y && q < nq && t < wl) yv = a.y[(int64_t)(q / K) * a.y_run_stride + ws + t];
            yb[((l >> 4) * kB + t) * kM + (l & 15)] = yv;
        }
        if (OPT) {
            float *hg = reinterpret_cast<float *>(lds + Lds::hg + buf * Lds::hg_bytes);
            for (int t = tid; t < kB; t += nthr) hg[t] = t < wl ? a.g01[ws + t] : 0.f;
        }
    };
    // shares of this wavefront of one tile's W X^T for one window -> LDS
    auto put_part = [&](const Geo<MT> &g, const f4 (&acc)[4]) __attribute__((always_inline)) {
        float *part = reinterpret_cast<float *>(lds + Lds::part);
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[(g.wave * kB + rb * 16 + 4 * g.lk + r) * kM + g.lr] = acc[rb][r];
    };
    // tile m's W' X_k^T = sum of the wavefronts' shares, fixed order, summed in float64
    auto sum_parts = [&](int tid, int m) __attribute__((always_inline)) {
        const float *part = reinterpret_cast<const float *>(lds + Lds::part);
        ST *q0d = reinterpret_cast<ST *>(lds + Lds::q0 + m * Lds::tile_s);
#pragma unroll
        for (int u = 0; u < kB * kM / (NW * kWave); ++u) {
            const int e = tid + u * NW * kWave;
            double sum = 0.0;
#pragma unroll
            for (int v = 0; v < NW; ++v) sum += (double)part[v * kB * kM + e];
            q0d[e] = (ST)sum;
        }
    };
    // ||w||^2 of tile m's learner lc as the last sweep measured it: 4 NW shares, fixed order
    auto measured_n2 = [&](int m, int lc) __attribute__((always_inline)) {
        const float *n2s = reinterpret_cast<const float *>(lds + Lds::n2) + m * NW * 4 * kM;
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < NW * 4; ++i) v += (double)n2s[i * kM + lc];
        return v;
    };

    // ---- per-learner state of the dependent rounds (wavefront m < MT: lane = 4 learner + quad lane) ----
    float eta = 0.f;
    double pmul = 1.0;          // scale of the iterates q0 was taken with: sigma of the state, then F of the window before
    double n2 = 0.0;            // ||w_k||^2 as the scalar identity carries it
    double n2_begin = 0.0;      // what the previous window's rounds started from
    bool proj_prev = true;      // whether they projected this learner (then n2 was reset to D^2 on the way)
    Hint hint{0.f, 0.f, 0.f};   // optimistic update: carried from round to round, window to window, call to call
    f4 V[RES ? NB : 1][MT];     // iterates in registers: the blocks kept_block() names, of every tile
    f4 accq[MT][4];             // this wavefront's shares of W_k X_{k+1}^T; tile 0's go to LDS at once, the others wait their turn
    {
        const Geo<MT> g = make_geo<MT>((int)threadIdx.x, a);
        const int q_ch = q_base + rounds_tile(g.wave) * kM + (g.lane >> 2);
        if (rounds_tile(g.wave) >= 0 && q_ch < nq) {
            eta = a.eta[q_ch % K];
            pmul = (double)a.sigma[q_ch];
            n2 = a.n2[q_ch] * pmul * pmul;                      // ||w||^2 of the iterate itself
            if (OPT) {
                const int ws0 = plan.start(w0);
                hint.ha = a.ha[q_ch];
                hint.hp = a.hp[q_ch];
                hint.x2p = ws0 == 0 ? a.x2last[0] : a.x2[ws0 - 1];
            }
        }
        if (RES) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int m = 0; m < MT; ++m) V[b][m] = ld_block(g, m, kept_block(g.wave, b));
        }
        // ---- prologue: the stored iterates times the rows of the first two windows -----------------
        f4 acc0[MT][4];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) { acc0[m][rb] = f4{0.f, 0.f, 0.f, 0.f}; accq[m][rb] = f4{0.f, 0.f, 0.f, 0.f}; }
        auto q_of = [&](const f4 (&vb)[MT], int blk) __attribute__((always_inline)) {
            f4 xr[4];
            ldq(g, 0, blk, xr);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
                        acc0[m][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xr[rb][r], vb[m][r], acc0[m][rb], 0, 0, 0);
            if (nw > 1) {
                ldq(g, 1, blk, xr);
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int rb = 0; rb < 4; ++rb)
                            accq[m][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xr[rb][r], vb[m][r], accq[m][rb], 0, 0, 0);
            }
        };
        if constexpr (RES) {
            static_for<NB>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value;
                const int blk = kept_block(g.wave, b);
                if (blk < nblk) q_of(V[b], blk);
            });
        } else {
            for (int i = 0, blk = nth_block(g.wave, 0); blk < nblk; blk = nth_block(g.wave, ++i)) {
                f4 vb[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) vb[m] = ld_block(g, m, blk);
                q_of(vb, blk);
            }
        }
        stage_chain_inputs(g.tid, NW * kWave, 0);
        {
            f4 gv[kGPer / 4];
            load_gram(g.tid, 0, gv);
            store_gram(g.tid, gv);
        }
        float *corr = reinterpret_cast<float *>(lds + Lds::corr);
        for (int e = g.tid; e < MT * kB * kM; e += NW * kWave) corr[e] = 0.f;
        // the shares of window 0 are summed here, tile by tile, so that those of window 1 can take their place
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            put_part(g, acc0[m]);
            __syncthreads();
            sum_parts(g.tid, m);
            __syncthreads();
        }
        if (nw > 1) put_part(g, accq[0]);
    }

#ifdef OCO_WIN_PROF
    unsigned long long prof_[8] = {0, 0, 0, 0, 0, 0, 0, 0}, last_ = wall_clock64();
#endif
    for (int k = 0; k <= nw; ++k) {
        int tid_w = (int)threadIdx.x;
        asm volatile("" : "+v"(tid_w));                          // see Geo
        const bool rounds = k < nw;                              // this iteration has dependent rounds (window k)
        const bool sweep = k >= 1;                               // ... and a sweep (window k - 1)
        const bool more = k + 1 < nw;                            // the sweep also takes W_k X_{k+1}^T
        // the cross Gram matrix of windows k - 1 and k as matrix operand, on its way across the barrier
        f4 gx[4];
        const int wave_w = __builtin_amdgcn_readfirstlane(tid_w >> 6);
        const bool corr_wave = rounds && sweep && wave_w < 4 * MT;   // four wavefronts per tile
        if (corr_wave) {
            const float *t = gxt + (int64_t)k * kB * kB + (wave_w & 3) * 1024 + (tid_w & 63) * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) gx[j] = *reinterpret_cast<const f4 *>(t + j * 256);
        }
        f4 gpre[kGPer / 4];
        const bool gram_now = rounds && k >= 1;                  // (window 0's table: prologue)
        if (gram_now) load_gram(tid_w, k, gpre);
        __syncthreads();                                         // (A) shares of W' X_k^T, -Bm_{k-1}, staged inputs in LDS
        PROF_T(0);
        if (gram_now) store_gram(tid_w, gpre);                   // (the rounds of window k - 1 are long done with theirs)
        if (rounds && k >= 1) {                                  // (window 0: summed in the prologue)
            sum_parts(tid_w, 0);
            if (MT > 1) {
                const Geo<MT> g1 = make_geo<MT>(tid_w, a);
#pragma unroll
                for (int m = 1; m < MT; ++m) {
                    __syncthreads();
                    put_part(g1, accq[m]);
                    __syncthreads();
                    sum_parts(tid_w, m);
                }
            }
        }
        if (corr_wave) {
            // corr[t][learner] = -sum_r Bm_{k-1}[r][learner] Gx[r][t], rows t = 16 (wave % 4) .. + 15, tile wave / 4
            const int m = wave_w >> 2, rbw = wave_w & 3;
            const float *bmp = reinterpret_cast<const float *>(lds + Lds::bm + ((k - 1) & 1) * Lds::bm_bytes + m * Lds::tile_f);
            const int lr = tid_w & 15, lk = (tid_w & 63) >> 4;
            f4 c = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int rs = 0; rs < 16; ++rs)
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(gx[rs >> 2][rs & 3], bmp[(rs * 4 + lk) * kM + lr], c, 0, 0, 0);
            float *corr = reinterpret_cast<float *>(lds + Lds::corr + m * Lds::tile_f);
#pragma unroll
            for (int r = 0; r < 4; ++r) corr[(rbw * 16 + 4 * lk + r) * kM + lr] = c[r];
        }
        __syncthreads();                                         // (B)
        PROF_T(1);
        const int tile_w = rounds_tile(wave_w);
        if (tile_w >= 0) {
            if (rounds) {
                const int lane = tid_w & 63;
                if (k >= 2) {
                    // ||w_{k-1}||^2 as the sweep of window k - 2 measured it against what the rounds of window
                    // k - 1 started from: the difference (float32 rounding of the sweeps) went through those
                    // rounds added to every squared norm, and every projection among them scaled it by f^2
                    // (to first order), so F_{k-1}^2 of it is still in the iterate and missing from n2.  The
                    // next projection then removes it from the iterate as well.
                    n2 = fma(measured_n2(tile_w, lane >> 2) - n2_begin, pmul * pmul, n2);
                    n2 = n2 > 0.0 ? n2 : 0.0;
                }
                n2_begin = n2;
                const double fscale = k == 0 ? pmul : 1.0;
                pmul = chain_window<LOSS, Lds, OPT>(lds, k & 1, tile_w, lane, plan.len(w0 + k), eta, (double)a.D, pmul, fscale,
                                                       n2, proj_prev, &hint);
            }
        } else {
            const int tid_o = other_index(wave_w) * kWave + (tid_w & 63), nthr_o = (NW - MT) * kWave;
            // beside the dependent rounds: the next window's labels and Gram table into the other buffer
            if (more) stage_chain_inputs(tid_o, nthr_o, k + 1);
            // ... and the predictions of window k - 1 to Z (a learner's rounds contiguous)
            if (sweep) {
                const int w = w0 + k - 1;
                const int ws = plan.start(w), wl = plan.len(w);
                const float *zb = reinterpret_cast<const float *>(lds + Lds::zb + ((k - 1) & 1) * Lds::zb_bytes);
                for (int e = tid_o; e < MT * kB * kM; e += nthr_o) {
                    const int l = e >> 6, t = e & 63;
                    const int q = q_base + l;
                    if (q < nq && t < wl)
                        a.Z[(int64_t)(q / K) * a.zl.zs_r + (int64_t)(q % K) * a.zl.zs_i + (int64_t)(ws + t) * a.zl.zs_t] =
                            zb[((l >> 4) * kB + t) * kM + (l & 15)];
                }
            }
        }
        PROF_T(2);
        asm volatile("" : "+v"(tid_w));
        const Geo<MT> g = make_geo<MT>(tid_w, a);
        const int lr = g.lr, lk = g.lk;

        // ---- sweep: (3) of window k - 1 and W_k X_{k+1}^T, block by block ------------------------------
        if (sweep) {
            const int wi = k - 1;
            const float *bml = reinterpret_cast<const float *>(lds + Lds::bm + (wi & 1) * Lds::bm_bytes);
            float bmr[MT][BMR ? 16 : 1];
            float F[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if (BMR) {
#pragma unroll
                    for (int rs = 0; rs < 16; ++rs) bmr[m][rs] = bml[m * kB * kM + (rs * 4 + lk) * kM + lr];
                }
                F[m] = reinterpret_cast<const float *>(lds + Lds::fv + (wi & 1) * Lds::fv_bytes)[m * kM + lr];
            }
            f4 acc[MT][4];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb) acc[m][rb] = f4{0.f, 0.f, 0.f, 0.f};
            float nn[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) nn[m] = 0.f;
            struct BlkIn { f4 xu[4]; f4 xq[4]; f4 vb[MT]; };
            const int wq = more ? k + 1 : k;                     // (no window after the last: any rows, unused)
            auto load_in = [&](BlkIn &in, int blk) __attribute__((always_inline)) {
                if constexpr (RES) {
                    if (blk < nblk) {
                        ldu(g, wi, blk, in.xu);
                        if (more) ldq(g, k + 1, blk, in.xq);
                    }
                } else {
                    // no branch around a load: a block past the end reads the last one again
                    const int b = blk < nblk ? blk : nblk - 1;
                    ldu(g, wi, b, in.xu);
                    ldq(g, wq, b, in.xq);
#pragma unroll
                    for (int m = 0; m < MT; ++m) in.vb[m] = ld_block_nb(g, m, b);
                }
            };
            auto compute = [&](BlkIn &in, f4 (&vreg)[MT], int blk) __attribute__((always_inline)) {
                f4 vb[MT], vo[MT];                               // per tile two chains of eight dependent instructions
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    vb[m] = RES ? vreg[m] : in.vb[m];
                    vo[m] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int r = 0; r < 4; ++r) vb[m][r] *= F[m];
                }
#pragma unroll
                for (int rs = 0; rs < 16; rs += 2)
#pragma unroll
                    for (int m = 0; m < MT; ++m) {
                        const float b0 = BMR ? bmr[m][BMR ? rs : 0] : bml[m * kB * kM + (rs * 4 + lk) * kM + lr];
                        const float b1 = BMR ? bmr[m][BMR ? rs + 1 : 0] : bml[m * kB * kM + ((rs + 1) * 4 + lk) * kM + lr];
                        vb[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(in.xu[rs >> 2][rs & 3], b0, vb[m], 0, 0, 0);
                        vo[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(in.xu[rs >> 2][(rs & 3) + 1], b1, vo[m], 0, 0, 0);
                    }
#pragma unroll
                for (int m = 0; m < MT; ++m) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) vb[m][r] += vo[m][r];
#pragma unroll
                    for (int r = 0; r < 4; ++r) nn[m] = fmaf(vb[m][r], vb[m][r], nn[m]);
                    if (RES) vreg[m] = vb[m]; else st_block_nb(g, m, blk, vb[m]);
                }
                if (more) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                            for (int m = 0; m < MT; ++m)
                                acc[m][rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(in.xq[rb][r], vb[m][r], acc[m][rb], 0, 0, 0);
                }
            };
            f4 none[MT];
            if constexpr (RES) {
                // The round rows of the next block are on their way while the matrix instructions of the
                // current block run.
                BlkIn in[2];
                load_in(in[0], kept_block(g.wave, 0));
                static_for<NB>([&](auto bc) __attribute__((always_inline)) {
                    constexpr int b = decltype(bc)::value;
                    const int blk = kept_block(g.wave, b);
                    if (b + 1 < NB) load_in(in[(b + 1) & 1], kept_block(g.wave, b + 1));
                    __builtin_amdgcn_sched_barrier(0);
                    if (blk < nblk) compute(in[b & 1], V[b], blk);
                    __builtin_amdgcn_sched_barrier(0);
                });
            } else if constexpr (NW == kNW16) {
                // One set of input registers: a block's loads are issued when the block before it is
                // done, and the other three wavefronts of the SIMD keep the matrix cores busy meanwhile.
                BlkIn in;
                for (int i = 0, blk = nth_block(g.wave, 0); blk < nblk; blk = nth_block(g.wave, ++i)) {
                    load_in(in, blk);
                    __builtin_amdgcn_sched_barrier(0);
                    compute(in, none, blk);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                // Two sets of input registers: the next block's loads are in flight during a block's
                // matrix instructions.  No load or store of the loop sits under a branch, so that every
                // wait leaves exactly the younger ones outstanding (the block's two stores and the eleven
                // loads of the next block).
                BlkIn in[2];
                int i = 0;
                load_in(in[0], nth_block(g.wave, 0));
                // (the loop is entered the way it is re-entered, with MT stores younger than the loads:
                // the wait at its head is computed from both and would otherwise drain the stores)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    *reinterpret_cast<f4 *>(misc + kMiscZeros + m * 2048 + g.tid * 4) = f4{0.f, 0.f, 0.f, 0.f};
                for (; nth_block(g.wave, i + 1) < nblk; i += 2) {
                    load_in(in[1], nth_block(g.wave, i + 1));
                    __builtin_amdgcn_sched_barrier(0);
                    compute(in[0], none, nth_block(g.wave, i));
                    __builtin_amdgcn_sched_barrier(0);
                    load_in(in[0], nth_block(g.wave, i + 2));
                    __builtin_amdgcn_sched_barrier(0);
                    compute(in[1], none, nth_block(g.wave, i + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (nth_block(g.wave, i) < nblk) compute(in[0], none, nth_block(g.wave, i));
            }
            PROF_T(4);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                reinterpret_cast<float *>(lds + Lds::n2)[m * NW * 4 * kM + (g.wave * 4 + lk) * kM + lr] = nn[m];
            if (more) {
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb) accq[m][rb] = acc[m][rb];
                put_part(g, accq[0]);
            }
        }
        PROF_T(5);
    }
#ifdef OCO_WIN_PROF
    if (threadIdx.x == OCO_WIN_PROF_TID && blockIdx.x == 0)
        for (int i = 0; i < 8; ++i) g_win_prof[i] = prof_[i];
#endif

    // ---- state out: the iterates themselves (scale 1) and their squared norms ---------------------
    {
        const Geo<MT> g = make_geo<MT>((int)threadIdx.x, a);
        if (RES) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int m = 0; m < MT; ++m) st_block(g, m, kept_block(g.wave, b), V[b][m]);
        }
        __syncthreads();
        const int q_ch = q_base + rounds_tile(g.wave) * kM + (g.lane >> 2);
        if (rounds_tile(g.wave) >= 0 && (g.lane & 3) == 0 && q_ch < nq) {
            a.sigma[q_ch] = 1.f;
            a.n2[q_ch] = measured_n2(rounds_tile(g.wave), g.lane >> 2);
            if (OPT) { a.ha[q_ch] = hint.ha; a.hp[q_ch] = hint.hp; }
        }
    }
}

// ---- the same windows with rows and iterates brought to LDS by wavefronts of their own -----------
// Four tiles of 16 learners per workgroup, two working wavefronts per tile (wavefront tau + 4 sigma:
// tile tau, blocks 2 s + sigma), and four wavefronts that only load.  All step through the blocks
// together, one barrier per step.  The loaders bring to a ring of three LDS stages the rows of
// the step's two blocks -- window k's in the lane order of (3), window k + 1's in that of (1) --
// which serve all four tiles (2 KB of rows from L2 per tile and block, in parts 3, where a wavefront that loads
// its own rows needs 8), and the eight blocks of iterates of the step; their registers are the
// prefetch buffer (the loads of four steps are on their way, in parts of three).  The working wavefronts read
// operands from LDS while matrix instructions run, and store the new block; they never wait for a memory instruction.  (On this hardware one counter per
// wavefront covers loads and stores alike and runs in issue order, so a wavefront that stores
// cannot wait for a younger load without also waiting for the acknowledgement of every older
// store, several microseconds here.)
// Windows are not overlapped here: sweep k (step (3) of window k, then W X^T for window k + 1)
// follows the dependent rounds of window k, which wavefront tau runs for tile tau; the inner
// products they start from are exact (no cross-Gram correction) and ||w||^2 is the sum of squares
// the sweep has just taken.  Wavefronts of the workgroup exchange data through LDS only, except
// that the loaders read iterates the others stored one sweep earlier (they wait for those stores
// once per window, after the dependent rounds); the barriers are therefore bare s_barrier
// instructions behind a wait for the LDS operations of the wavefront (__syncthreads() would also
// wait for every store's acknowledgement).
// Measured with float32 rows on c4 (one workgroup per compute unit, 128 steps per window): 1.07 us per step with the
// loads switched off against 0.85 us of matrix instructions, 1.35 to 1.45 us with them, whether the
// loads go through registers or straight to LDS and whatever their distance; the dependent rounds
// (not overlapped) and the hand-over between the phases add 35 us per window.
// Long calls of whole blocks (parts_pay) are the PARTS form: rows and iterates enter the matrix instructions as three
// bfloat16 parts (split2).  The rows are split once per launch
// (dense_tile_split_kernel), -Bm once per window, an iterate's block when it has been updated; sums and the iterates
// themselves stay float32.  Per block 24 instructions of 16 clocks in place of 32 of 32, for 6 KB of rows per window and
// block instead of 4.  Error against float64 on c4: 4.9e-7, with float32 instructions 6.9e-7.
// Measured on c4 as above, us per step: 1.02; 0.75 with the loads switched off (LDS reads, matrix and vector instructions), 0.84 with either the
// rows or the iterates loaded alone, as long without matrix instructions as with them.  Of a window 131 us are the sweep, 10.7 the
// dependent rounds, 3.7 inputs and shares.  What bounds it is the iterates' way through HBM, with the rows (from L2) beside it: by
// the byte counters the sweep moves 4.5 TB/s, 0.86 of what a device copy does, the matrix cores are busy a third of the time and
// LDS 0.36.  The iterates are loaded and stored with the streaming hint, both or
// neither (one of them: 10 ms per step worse), and lie in blocks (below).  Workgroups of an XCD held to one pace
// by a counter: 10 ms worse; a different first block per XCD or workgroup: no difference; rows and iterates on loading
// wavefronts of their own: no better with the hint, 17 ms worse without; four steps ahead instead of three: spills.
constexpr int kQT = 4, kQS = 2;              // tiles per workgroup, working wavefronts per tile
constexpr int kQW = kQT * kQS;               // working wavefronts; wavefront kQW loads
constexpr int kQStages = 3;
constexpr int kQL = 4;                       // loading wavefronts
// steps of loads each of them keeps in registers; steps are walked in multiples of the second (of kQStages and of the first)
template <bool PARTS> constexpr int kQSets = PARTS ? 3 : 4;
template <bool PARTS> constexpr int kQUnroll = PARTS ? 6 : 12;
static_assert(kQUnroll<true> % kQStages == 0 && kQUnroll<true> % kQSets<true> == 0 && kQUnroll<false> % kQStages == 0 &&
              kQUnroll<false> % kQSets<false> == 0 && kQUnroll<false> % 2 == 0, "stages and register sets are compile-time constants");
template <bool PARTS> struct LdsQ {
    using G = double;
    using S = float;
    static constexpr int g_reads = 0;
    static constexpr bool carry_norm = false;
    static constexpr bool has_corr = false;
    static constexpr int gd_bytes = kB * 4 * kGStride * 8;
    static constexpr int tile_f = kB * kM * 4, tile_s = tile_f;
    static constexpr int yb_bytes = kQT * tile_f, zb_bytes = kQT * tile_f, bm_bytes = kQT * tile_f, fv_bytes = kQT * kM * 4;
    static constexpr int blk_bytes = (PARTS ? kSplitFloats : kTileFloats) * 4;   // a block's rows of one window
    static constexpr int rows_bytes = kQS * 2 * blk_bytes;         // per step and block: rows for (3), rows for (1)
    static constexpr int stage_bytes = rows_bytes + kQW * 1024;    // ... and a block of iterates per working wavefront
    static constexpr int gd = 0;
    static constexpr int yb = gd + gd_bytes;
    static constexpr int fv = yb + yb_bytes + (PARTS ? 0 : zb_bytes + bm_bytes);
    static constexpr int n2 = fv + fv_bytes;                       // float [kQT][kQS * 4][16]: shares of ||w||^2
    static constexpr int hg = n2 + kQT * kQS * 4 * kM * 4;         // float [64]: <x_{t-1}, x_t> of the window's rounds (optimistic update)
    static constexpr int hg_bytes = kB * 4;
    static constexpr int ring = hg + hg_bytes;
    // between two sweeps the ring's space holds the shares of W X^T, [kQS][kQT][64][16] (share 0
    // becomes the sum), and the a_t and f_t of the dependent rounds
    static constexpr int q0 = ring;
    static constexpr int part_bytes = kQT * tile_f;
    static constexpr int st = ring + kQS * part_bytes;
    static constexpr int fl = st + kQT * tile_f;
    // ... and, beside the longer rows of the parts, the predictions and -Bm, which are read before the barrier that lets the
    // loaders write stage 1
    static constexpr int zb = PARTS ? fl + kQT * tile_s : yb + yb_bytes;
    static constexpr int bm = zb + zb_bytes;
    static constexpr int corr = 0;                                 // (unused)
    static constexpr int total = ring + kQStages * stage_bytes;
};
template <bool PARTS> constexpr bool lds_q_ok()
{
    using L = LdsQ<PARTS>;
    return L::fl + kQT * L::tile_s <= L::total && L::bm + L::bm_bytes <= L::total && L::total <= 160 * 1024;
}
static_assert(lds_q_ok<false>() && lds_q_ok<true>(), "LDS of a gfx950 compute unit");
static_assert(LdsQ<true>::zb >= LdsQ<true>::ring + LdsQ<true>::stage_bytes, "stage 0 is written while -Bm and the predictions are read");

// The iterates of a tile of 16 learners, in place from rows [16][d] to blocks of 16 coordinates [d / 16][64][4] as a wavefront
// of the sweep loads and stores them (lane l: coordinates 4 (l / 16) .. of learner l % 16), or back: a block is then 1 KB of
// memory in one piece instead of sixteen 64-byte pieces d floats apart.  One workgroup holds the tile in registers in between.
// c4 with rows in parts: 65.6 ms per step from rows, 59.1 from blocks (0.1 ms each way); with float32 rows 68.4 and 65.4.
constexpr int kBlocksMaxD = 4096;
template <bool BACK> __global__ void __launch_bounds__(1024) tile_blocks_kernel(float *V, int d)
{
    f4 *v = reinterpret_cast<f4 *>(V + (int64_t)blockIdx.x * kM * d);
    const int n = kM * d / 4, d4 = d / 4;
    constexpr int N = kM * kBlocksMaxD / 4 / 1024;
    f4 o[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int e = (int)threadIdx.x + i * 1024;
        if (e < n) o[i] = v[e];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // everything is in registers before the first store
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int e = (int)threadIdx.x + i * 1024;
        if (e >= n) continue;
        if (BACK) v[(e & 15) * d4 + (e >> 6) * 4 + ((e >> 4) & 3)] = o[i];
        else v[(e % d4 >> 2) * 64 + (e % d4 & 3) * 16 + e / d4] = o[i];
    }
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// -Bm of a lane's learner: as float32, round 4 rs + l / 16, or in parts, rounds 32 s + 8 (l / 16) ..
struct StepsF { float v[16]; };
struct StepsP { u4 p[2][3]; };

// PARTS: rows and iterates as bfloat16 parts (such launches are timed under the name dense_window_parts_kernel)
template <int LOSS, bool OPT, bool PARTS>
__global__ void __launch_bounds__((kQW + kQL) * kWave) dense_window_shared_kernel(const DenseArgs a, const float *gram, const float *gxt,
                                                                               const float *xq, const float *xu, float *misc,
                                                                               WinPlanD plan, int w0, int nw)
{
    // (gxt: no cross Gram matrix here; not null: the iterates lie in blocks, see tile_blocks_kernel)
    const bool blocked = PARTS && gxt != nullptr;
    const int vstep = blocked ? 16 * kM : 16;                    // from a block of a lane's learner to the next
    using Lds = LdsQ<PARTS>;
    using Steps = std::conditional_t<PARTS, StepsP, StepsF>;
    constexpr int SETS = kQSets<PARTS>, UNROLL = kQUnroll<PARTS>;
    constexpr int NC = Lds::blk_bytes / 1024;                    // 16-byte loads per lane and block of rows
    constexpr int NT = kQW * kWave;                              // working threads
    extern __shared__ __align__(16) char lds[];
    const int d = a.d, K = a.K;
    const int nq = a.R * K;
    const int nblk = (d + 15) / 16;
    const int nstep = (nblk + kQS - 1) / kQS;
    const int npad = (nstep + UNROLL - 1) / UNROLL * UNROLL;   // steps every wavefront walks
    const int q_base = (int)blockIdx.x * kQT * kM;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool loader = wave >= kQW;
    const int tau = wave & (kQT - 1), sg = (wave / kQT) & (kQS - 1);
    const int lr = lane & 15, lk = lane >> 4;

    // dependent rounds: wavefront m < kQT, lane = 4 learner + quad lane
    float eta = 0.f;
    double sigma0 = 1.0, n2_state = 0.0;
    Hint hint{0.f, 0.f, 0.f};   // optimistic update: carried from round to round, window to window, call to call
    {
        const int q_ch = q_base + wave * kM + (lane >> 2);
        if (wave < kQT && q_ch < nq) {
            eta = a.eta[q_ch % K];
            sigma0 = (double)a.sigma[q_ch];
            n2_state = a.n2[q_ch] * sigma0 * sigma0;
            if (OPT) {
                const int ws0 = plan.start(w0);
                hint.ha = a.ha[q_ch];
                hint.hp = a.hp[q_ch];
                hint.x2p = ws0 == 0 ? a.x2last[0] : a.x2[ws0 - 1];
            }
        }
    }
    auto measured_n2 = [&](int m, int lc) __attribute__((always_inline)) {
        const float *n2s = reinterpret_cast<const float *>(lds + Lds::n2) + m * kQS * 4 * kM;
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < kQS * 4; ++i) v += (double)n2s[i * kM + lc];
        return v;
    };
#ifdef OCO_WIN_PROF
    unsigned long long prof_[8] = {0, 0, 0, 0, 0, 0, 0, 0}, last_ = wall_clock64();
#endif

    struct Regs { f4 r[NC + 2]; };
    Regs rg[SETS];                                               // loaders: SETS steps of loads (the prefetch buffer)
    // The loaders' side of a sweep: rows for (3) from window wu of the piece, rows for (1) from window wq.
    // `first`: the loads of the first SETS steps are issued here; otherwise they were issued at the end of
    // the sweep before (nwu >= 0: issue those of the next sweep, rows from windows nwu / nwq), so that
    // they travel while the dependent rounds run.
    auto load_sweep = [&](int wu, int wq, bool first, int nwu, int nwq) __attribute__((always_inline)) {
        // (what a lane is, from an index the compiler cannot see through: kept across the dependent rounds it would be
        // spilled, and every reload in the loop would wait for all the loads on their way)
        int tid_l = (int)threadIdx.x;
        asm volatile("" : "+v"(tid_l));
        const int lane = tid_l & 63, lr = lane & 15, lk = lane >> 4;
        // the learners whose blocks this lane loads, tile by tile
        const float *vr[2];
        bool vok[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int q = q_base + (2 * ((wave - kQW) >> 1) + m) * kM + lr;
            vok[m] = q < nq;
            vr[m] = a.V + (blocked ? (int64_t)(vok[m] ? q / kM : 0) * kM * d + 4 * lane : (int64_t)(vok[m] ? q : 0) * d + 4 * lk);
        }
        // loader j: block kQS s + (j & 1) of step s; j < 2 its rows for (3) and the iterates of tiles 0, 1,
        // j >= 2 its rows for (1) and the iterates of tiles 2, 3
        const int L = (wave - kQW) & 1, part = (wave - kQW) >> 1;
        auto fetch_of = [&](int fu, int fq, int step, Regs &o) __attribute__((always_inline)) {
            const int sc = step < nstep ? step : nstep - 1;
            int blk = sc * kQS + L;
            blk = blk < nblk ? blk : nblk - 1;                   // (rows past the last block: loaded again, not used)
            const float *src = (part == 0 ? xu + ((int64_t)fu * nblk + blk) * (Lds::blk_bytes / 4)
                                          : xq + ((int64_t)fq * nblk + blk) * (Lds::blk_bytes / 4)) + lane * 4;
#pragma unroll
            for (int c = 0; c < NC; ++c) o.r[c] = *reinterpret_cast<const f4 *>(src + c * 256);
            const int vblk = step * kQS + L;
            const bool bok = step < nstep && vblk < nblk && vblk * 16 + 4 * lk < d;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const f4 *vp = reinterpret_cast<const f4 *>((bok && vok[m]) ? vr[m] + (int64_t)vblk * vstep : misc);
                o.r[NC + m] = PARTS ? __builtin_nontemporal_load(vp) : *vp;
            }
        };
        auto fetch = [&](int step, Regs &o) __attribute__((always_inline)) { fetch_of(wu, wq, step, o); };
        auto put = [&](int stage, const Regs &o) __attribute__((always_inline)) {
            char *st = lds + Lds::ring + stage * Lds::stage_bytes + lane * 16;
#pragma unroll
            for (int c = 0; c < NC; ++c) *reinterpret_cast<f4 *>(st + (2 * L + part) * Lds::blk_bytes + c * 1024) = o.r[c];
#pragma unroll
            for (int m = 0; m < 2; ++m) *reinterpret_cast<f4 *>(st + Lds::rows_bytes + (L * kQT + 2 * part + m) * 1024) = o.r[NC + m];
        };
        // Phase p (up to barrier p): step p's operands from registers to stage p % 3, then the loads of step
        // p + SETS into the registers they came from (the registers are the prefetch buffer: SETS steps of
        // loads are on their way).  After barrier p the working wavefronts read stage p while they work step
        // p - 1; the stage was last read two phases earlier.
        if (first) {
#pragma unroll
            for (int s0 = 0; s0 < SETS; ++s0) fetch(s0, rg[s0]);
        }
        put(0, rg[0]);
        fetch(SETS, rg[0]);
        lds_barrier();
        for (int sb = 0; sb < npad; sb += UNROLL) {
            static_for<UNROLL>([&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                put((u + 1) % kQStages, rg[(u + 1) % SETS]);
                fetch(sb + u + 1 + SETS, rg[(u + 1) % SETS]);
                lds_barrier();
            });
        }
        // (the blocks of iterates of the next sweep's first steps were stored at the start of this one: the
        // working wavefronts have waited for those stores before the last barrier above)
        if (nwu >= 0) {
#pragma unroll
            for (int s0 = 0; s0 < SETS; ++s0) fetch_of(nwu, nwq, s0, rg[s0]);
        }
        lds_barrier();
        lds_barrier();
        lds_barrier();
    };

    // Labels and Gram table of the next window: the working wavefronts that do not run dependent rounds
    // (kQT .. kQW - 1) load them into registers beside those rounds (whose LDS copies are still in use) and
    // write them to LDS once the rounds are done.
    constexpr int kNPre = (kQW - kQT) * kWave;                  // threads that stage
    constexpr int kGPer = kB * kB / kNPre, kYPer = kQT * kM * kB / kNPre;
    f4 gpre[kGPer / 4];
    float ypre[kYPer];
    float hgpre = 0.f;                                           // (optimistic update: <x_{t-1}, x_t> of one round)
    auto load_next = [&](int wi) __attribute__((always_inline)) {
        const int tp = tid - kQT * kWave;
        const int w = w0 + wi;
        const int ws = plan.start(w), wl = plan.len(w);
        const float *gsrc = gram + (int64_t)wi * kB * kB + tp * kGPer;
#pragma unroll
        for (int i = 0; i < kGPer / 4; ++i) gpre[i] = *reinterpret_cast<const f4 *>(gsrc + 4 * i);
#pragma unroll
        for (int i = 0; i < kYPer; ++i) {
            const int e = tp + i * kNPre, l = e >> 6, t = e & 63;
            const int q = q_base + l;
            const bool ok = a.y && q < nq && t < wl;              // (no label: a zero word)
            ypre[i] = *(ok ? a.y + (int64_t)(q / K) * a.y_run_stride + ws + t : misc);
        }
        if (OPT) hgpre = *((tp < kB && tp < wl) ? a.g01 + ws + tp : misc);
    };
    auto store_next = [&]() __attribute__((always_inline)) {
        const int tp = tid - kQT * kWave;
        double *gd = reinterpret_cast<double *>(lds + Lds::gd);
        const int t = (tp * kGPer) >> 6, t2b = (tp * kGPer) & 63;
#pragma unroll
        for (int i = 0; i < kGPer; ++i) {
            const int t2 = t2b + i;
            const float v = gpre[i >> 2][i & 3];
            gd[(t * 4 + (i & 3)) * kGStride + (t2 >> 2)] = t2 > t ? (double)v : 0.0;
            if (t2 == t) *reinterpret_cast<float *>(gd + t * 4 * kGStride + 16) = v;
        }
        float *yb = reinterpret_cast<float *>(lds + Lds::yb);
#pragma unroll
        for (int i = 0; i < kYPer; ++i) {
            const int e = tp + i * kNPre, l = e >> 6, t = e & 63;
            yb[((l >> 4) * kB + t) * kM + (l & 15)] = ypre[i];
        }
        if (OPT && tp < kB) reinterpret_cast<float *>(lds + Lds::hg)[tp] = hgpre;
    };

    // The working wavefronts' side.  F and -Bm of this lane's learner; do_q: take the shares of W X^T.  stage_next:
    // first write the staged labels and Gram table to LDS; flush_prev >= 0: write the predictions of window flush_prev to Z.
    auto sweep = [&](auto stager, bool do_q, float F, const Steps &bmr, bool stage_next, int flush_prev)
        __attribute__((always_inline)) {
        int tid_s = (int)threadIdx.x;                            // (see load_sweep)
        asm volatile("" : "+v"(tid_s));
        const int tid = tid_s, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
        const int q_sw = q_base + tau * kM + lr;                 // this lane's learner
        const bool q_ok = q_sw < nq;
        float *vrow = a.V + (blocked ? (int64_t)(q_ok ? q_sw / kM : 0) * kM * d + 4 * lane : (int64_t)(q_ok ? q_sw : 0) * d + 4 * lk);
        float *sink = misc + kMiscZeros + (tid & (NT - 1)) * 4;
        if (flush_prev >= 0) {
            const int w = w0 + flush_prev;
            const int ws = plan.start(w), wl = plan.len(w);
            const float *zb = reinterpret_cast<const float *>(lds + Lds::zb);
            for (int e = tid; e < kQT * kM * kB; e += NT) {
                const int l = e >> 6, t = e & 63;               // a learner's 64 rounds are contiguous in Z
                const int q = q_base + l;
                if (q < nq && t < wl)
                    a.Z[(int64_t)(q / K) * a.zl.zs_r + (int64_t)(q % K) * a.zl.zs_i + (int64_t)(ws + t) * a.zl.zs_t] =
                        zb[((l >> 4) * kB + t) * kM + (l & 15)];
            }
        }
        if constexpr (decltype(stager)::value) {
            if (stage_next) store_next();
        }
        f4 acc[4];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[rb] = f4{0.f, 0.f, 0.f, 0.f};
        float nn = 0.f;
        PROF_T(1);
        // all but the seven youngest stores acknowledged means those of the first SETS steps, which the loaders read
        // again right after the sweep, where there are enough of them
        const bool many = nstep > SETS + 8;
        auto wait_stores = [&](int step) __attribute__((always_inline)) {
            if (step == npad - 1) {
                if (many) asm volatile("s_waitcnt vmcnt(7)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        };
        if constexpr (PARTS) {
            // A step's operands of (3) and its block of iterates come from LDS while the matrix instructions of the
            // step before run, those of (1) while its own of (3) do.
            u4 ux[2][3];
            f4 vin;
            auto read_u = [&](int stage) __attribute__((always_inline)) {
                const char *stg = lds + Lds::ring + stage * Lds::stage_bytes;
                vin = *reinterpret_cast<const f4 *>(stg + Lds::rows_bytes + (sg * kQT + tau) * 1024 + lane * 16);
#pragma unroll
                for (int c = 0; c < NC; ++c) ux[c & 1][c >> 1] = *reinterpret_cast<const u4 *>(stg + 2 * sg * Lds::blk_bytes + c * 1024 + lane * 16);
            };
            lds_barrier();                                       // the loader has stage 0 complete
            read_u(0);
            for (int sb = 0; sb < npad; sb += UNROLL) {
                static_for<UNROLL>([&](auto uc) __attribute__((always_inline)) {
                    constexpr int u = decltype(uc)::value;
                    const int step = sb + u;
                    const int blk = step * kQS + sg;
                    wait_stores(step);
                    lds_barrier();                                   // stage step + 1 complete; stage step - 1 is not read any more
                    u4 q12[4], q3[2];
                    {
                        const char *qs = lds + Lds::ring + (u % kQStages) * Lds::stage_bytes + (2 * sg + 1) * Lds::blk_bytes + lane * 16;
#pragma unroll
                        for (int c = 0; c < 4; ++c) q12[c] = *reinterpret_cast<const u4 *>(qs + c * 1024);
#pragma unroll
                        for (int c = 0; c < 2; ++c) q3[c] = *reinterpret_cast<const u4 *>(qs + (4 + c) * 1024);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    const bool active = step < nstep && blk < nblk;  // wavefront-uniform
                    f4 vb = vin, vo = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int r = 0; r < 4; ++r) vb[r] *= F;
                    // the small products first, apart from the large ones
                    vo = mfma_bf16(ux[0][2], bmr.p[0][0], vo);
                    vb = mfma_bf16(ux[0][0], bmr.p[0][0], vb);
                    vo = mfma_bf16(ux[0][0], bmr.p[0][2], vo);
                    vb = mfma_bf16(ux[1][0], bmr.p[1][0], vb);
                    vo = mfma_bf16(ux[1][2], bmr.p[1][0], vo);
                    vo = mfma_bf16(ux[1][0], bmr.p[1][2], vo);
                    vo = mfma_bf16(ux[0][1], bmr.p[0][1], vo);
                    vo = mfma_bf16(ux[1][1], bmr.p[1][1], vo);
                    vo = mfma_bf16(ux[0][1], bmr.p[0][0], vo);
                    vo = mfma_bf16(ux[0][0], bmr.p[0][1], vo);
                    vo = mfma_bf16(ux[1][1], bmr.p[1][0], vo);
                    vo = mfma_bf16(ux[1][0], bmr.p[1][1], vo);
                    __builtin_amdgcn_sched_barrier(0);
                    read_u((u + 1) % kQStages);
#pragma unroll
                    for (int r = 0; r < 4; ++r) vb[r] += vo[r];
                    if (active) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) nn = fmaf(vb[r], vb[r], nn);
                        {
                            const bool ok = q_ok && blk * 16 + 4 * lk < d;
                            float *dst = ok ? vrow + (int64_t)blk * vstep : sink;
                            __builtin_nontemporal_store(vb, reinterpret_cast<f4 *>(dst));   // (streams: the rows stay in L2)
                        }
                        if (do_q) {
                            unsigned a1, a2, a3, b1, b2, b3;
                            split2(vb[0], vb[1], a1, a2, a3);
                            split2(vb[2], vb[3], b1, b2, b3);
                            const u4 w11 = u4{a1, b1, a1, b1}, w22 = u4{a2, b2, a2, b2}, w31 = u4{a3, b3, a1, b1};
#pragma unroll
                            for (int rb = 0; rb < 4; ++rb) {
                                const u4 x13 = u4{q12[rb][0], q12[rb][1], q3[rb >> 1][2 * (rb & 1)], q3[rb >> 1][2 * (rb & 1) + 1]};
                                acc[rb] = mfma_bf16(x13, w31, acc[rb]);
                            }
#pragma unroll
                            for (int rb = 0; rb < 4; ++rb) acc[rb] = mfma_bf16(q12[rb], w22, acc[rb]);
#pragma unroll
                            for (int rb = 0; rb < 4; ++rb) acc[rb] = mfma_bf16(q12[rb], w11, acc[rb]);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
        } else {
            // Two sets of operand registers: while the matrix instructions of step r - 1 run, the
            // operands of step r come from LDS (the eight wavefronts would otherwise all read right
            // after the barrier, 72 KB through the LDS port with the matrix cores idle).
            struct In { f4 xu[4], xq[4], vb; };
            In in[2];
            auto read_stage = [&](int stage, In &o) __attribute__((always_inline)) {
                const char *stg = lds + Lds::ring + stage * Lds::stage_bytes;
                const char *rows = stg + 2 * sg * Lds::blk_bytes + lane * 16;
                o.vb = *reinterpret_cast<const f4 *>(stg + Lds::rows_bytes + (sg * kQT + tau) * 1024 + lane * 16);
#pragma unroll
                for (int c = 0; c < 4; ++c) o.xu[c] = *reinterpret_cast<const f4 *>(rows + c * 1024);
#pragma unroll
                for (int c = 0; c < 4; ++c) o.xq[c] = *reinterpret_cast<const f4 *>(rows + Lds::blk_bytes + c * 1024);
            };
            lds_barrier();                                       // the loader has stage 0 complete
            read_stage(0, in[0]);
            for (int sb = 0; sb < npad; sb += 2 * kQStages) {
                static_for<2 * kQStages>([&](auto uc) __attribute__((always_inline)) {
                    constexpr int u = decltype(uc)::value;
                    const int step = sb + u;
                    const int blk = step * kQS + sg;
                    wait_stores(step);
                    lds_barrier();                               // stage step + 1 complete, own reads of stage step done
                    read_stage((u + 1) % kQStages, in[(u + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    const bool active = step < nstep && blk < nblk;  // wavefront-uniform
                    if (active) {
                        In &c = in[u & 1];
                        f4 vb = c.vb;
                        f4 vo = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int r = 0; r < 4; ++r) vb[r] *= F;
#pragma unroll
                        for (int rs = 0; rs < 16; rs += 2) {
                            vb = __builtin_amdgcn_mfma_f32_16x16x4f32(c.xu[rs >> 2][rs & 3], bmr.v[rs], vb, 0, 0, 0);
                            vo = __builtin_amdgcn_mfma_f32_16x16x4f32(c.xu[rs >> 2][(rs & 3) + 1], bmr.v[rs + 1], vo, 0, 0, 0);
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) vb[r] += vo[r];
#pragma unroll
                        for (int r = 0; r < 4; ++r) nn = fmaf(vb[r], vb[r], nn);
                        {
                            const bool ok = q_ok && blk * 16 + 4 * lk < d;
                            float *dst = ok ? vrow + blk * 16 : sink;
                            *reinterpret_cast<f4 *>(dst) = vb;
                        }
                        if (do_q) {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
#pragma unroll
                                for (int rb = 0; rb < 4; ++rb)
                                    acc[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.xq[rb][r], vb[r], acc[rb], 0, 0, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
        }
        PROF_T(2);
        lds_barrier();                                           // every wavefront is done with the ring
        {
            float *part = reinterpret_cast<float *>(lds + Lds::q0 + sg * Lds::part_bytes + tau * Lds::tile_f);
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[(rb * 16 + 4 * lk + r) * kM + lr] = acc[rb][r];
            reinterpret_cast<float *>(lds + Lds::n2)[(tau * kQS * 4 + sg * 4 + lk) * kM + lr] = nn;
        }
        lds_barrier();
        // the two shares of every tile's W X^T, summed in place
        if (do_q) {
            float *p0 = reinterpret_cast<float *>(lds + Lds::q0);
            const float *p1 = reinterpret_cast<const float *>(lds + Lds::q0 + Lds::part_bytes);
#pragma unroll
            for (int i = 0; i < kQT * kB * kM / NT; ++i) p0[tid + i * NT] += p1[tid + i * NT];
        }
        lds_barrier();
        PROF_T(3);
    };

    // Three programs with the same sequence of barriers, one per kind of wavefront, so that what one kind
    // keeps in registers across the window loop (the loaders' prefetch buffer, the staged inputs, the state of
    // the dependent rounds) is not live in the code of the others.
    // CHAIN: wavefronts 0 .. kQT - 1 run the dependent rounds of their tile; the other working wavefronts
    // stage the next window's labels and Gram table meanwhile.
    auto worker = [&](auto chain_tag) __attribute__((always_inline)) {
        constexpr bool CHAIN = decltype(chain_tag)::value;
        using Stager = std::integral_constant<bool, !CHAIN>;
        {
            // the stored iterates times the rows of the first window: a sweep whose step changes nothing
            const Steps zero{};
            if constexpr (!CHAIN) load_next(0);
            sweep(Stager{}, true, 1.f, zero, true, -1);
        }
        for (int k = 0; k < nw; ++k) {
            const bool more = k + 1 < nw;
            if constexpr (CHAIN) {
                double n2 = k == 0 ? n2_state : measured_n2(wave, lane >> 2);
                const double scale = k == 0 ? sigma0 : 1.0;
                bool projected;
                (void)chain_window<LOSS, Lds, OPT>(lds, 0, wave, lane, plan.len(w0 + k), eta, (double)a.D, scale, scale, n2, projected,
                                                   &hint);
            } else {
                if (more) load_next(k + 1);
            }
            PROF_T(0);
            // the iterates the last sweep stored are read by the loaders in the next one
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();
            PROF_T(4);
            Steps bmr;
            const float *bml = reinterpret_cast<const float *>(lds + Lds::bm + tau * Lds::tile_f) + lr;
            if constexpr (PARTS) {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int r = 32 * s2 + 8 * lk + 2 * j;
                        unsigned p1, p2, p3;
                        split2(bml[r * kM], bml[(r + 1) * kM], p1, p2, p3);
                        bmr.p[s2][0][j] = p1; bmr.p[s2][1][j] = p2; bmr.p[s2][2][j] = p3;
                    }
            } else {
#pragma unroll
                for (int rs = 0; rs < 16; ++rs) bmr.v[rs] = bml[(rs * 4 + lk) * kM];
            }
            const float F = reinterpret_cast<const float *>(lds + Lds::fv)[tau * kM + lr];
            sweep(Stager{}, more, F, bmr, more, k);
        }
    };
    if (loader) {
        load_sweep(0, 0, true, 0, nw > 1 ? 1 : 0);
        for (int k = 0; k < nw; ++k) {
            const bool more = k + 1 < nw;
            lds_barrier();
            load_sweep(k, more ? k + 1 : k, false, more ? k + 1 : -1, k + 2 < nw ? k + 2 : k + 1);
        }
    } else if (wave < kQT) {
        worker(std::true_type{});
    } else {
        worker(std::false_type{});
    }
#ifdef OCO_WIN_PROF
    if (threadIdx.x == 0 && blockIdx.x == 0)
        for (int i = 0; i < 8; ++i) g_win_prof[i] = prof_[i];
#endif
    // ---- state out: the iterates themselves (scale 1) and their squared norms ----------------------
    {
        const int q_ch = q_base + wave * kM + (lane >> 2);
        if (wave < kQT && (lane & 3) == 0 && q_ch < nq) {
            a.sigma[q_ch] = 1.f;
            a.n2[q_ch] = measured_n2(wave, lane >> 2);
            if (OPT) { a.ha[q_ch] = hint.ha; a.hp[q_ch] = hint.hp; }
        }
    }
}

using WindowKernel = void (*)(const DenseArgs, const float *, const float *, const float *, const float *, float *, WinPlanD, int,
                              int);

// mode 0: iterates in registers (8 wavefronts, one tile); 1: streamed, two tiles per workgroup
// (8 wavefronts); 2: streamed, one tile, 16 wavefronts; 3: four tiles, loading wavefronts; 4: iterates
// of two tiles in registers (8 wavefronts, d <= 1024)
// (opt: the optimistic update, built into the three kernels the launcher picks by itself)
template <int LOSS> WindowKernel pick_window_kernel(int nblk, int mode, bool parts, bool opt, int *waves, int *tiles, int *lds_bytes)
{
    if (mode == 3) {
        *waves = kQW + kQL; *tiles = kQT; *lds_bytes = parts ? LdsQ<true>::total : LdsQ<false>::total;
        if constexpr (LOSS != 0) {                               // (the linear loss: see parts_pay)
            if (parts) return opt ? dense_window_shared_kernel<LOSS, true, true> : dense_window_shared_kernel<LOSS, false, true>;
        }
        return opt ? dense_window_shared_kernel<LOSS, true, false> : dense_window_shared_kernel<LOSS, false, false>;
    }
    if (mode == 4) {
        *waves = kNW8; *tiles = 2; *lds_bytes = LdsT<kNW8, 2>::total;
        if (opt) return dense_window_kernel<LOSS, 9, true, kNW8, 2, true>;
        return dense_window_kernel<LOSS, 9, true, kNW8, 2>;
    }
    if (opt) {
        *waves = kNW8; *tiles = 2; *lds_bytes = LdsT<kNW8, 2>::total;
        return dense_window_kernel<LOSS, 1, false, kNW8, 2, true>;
    }
    if (mode == 0) {
        *waves = kNW8; *tiles = 1; *lds_bytes = LdsT<kNW8, 1>::total;
        if (nblk <= 8 * kNW8) return dense_window_kernel<LOSS, 8, true, kNW8, 1>;
        return dense_window_kernel<LOSS, 32, true, kNW8, 1>;
    }
    if (mode == 1) {
        *waves = kNW8; *tiles = 2; *lds_bytes = LdsT<kNW8, 2>::total;
        return dense_window_kernel<LOSS, 1, false, kNW8, 2>;
    }
    *waves = kNW16; *tiles = 1; *lds_bytes = LdsT<kNW16, 1>::total;
    return dense_window_kernel<LOSS, 1, false, kNW16, 1>;
}

// scratch: Gram and cross Gram matrices of the windows of a piece, then the two tiled copies of its rows
struct Scratch {
    int64_t piece_windows;      // windows per launch
    size_t gram_floats, tile_floats;
    size_t total_floats() const { return 2 * gram_floats + 2 * tile_floats + kMiscFloats; }
};
Scratch scratch_layout(int64_t n_max, int64_t d)
{
    const int64_t nblk = (d + 15) / 16;
    const int64_t win_bytes = nblk * kTileFloats * (int64_t)sizeof(float);
    Scratch sc;
    sc.piece_windows = std::max<int64_t>(1, std::min<int64_t>(kPieceBytes / win_bytes, n_max / kB + 2));
    sc.gram_floats = (size_t)sc.piece_windows * kB * kB;
    sc.tile_floats = (size_t)sc.piece_windows * nblk * kTileFloats;
    return sc;
}

}  // namespace

#ifdef OCO_WIN_PROF
extern "C" int oco_debug_win_prof(unsigned long long *out)
{
    return (int)hipMemcpyFromSymbol(out, HIP_SYMBOL(g_win_prof), sizeof(unsigned long long) * 8);
}
#endif

size_t dense_window_scratch_floats(int64_t n_max, int64_t d) { return scratch_layout(n_max, d).total_floats(); }
size_t dense_gram_bytes(int64_t n_max, int64_t d) { return scratch_layout(n_max, d).total_floats() * sizeof(float); }

bool dense_window_supported(const DenseArgs &a)
{
    // a shared stream whose rows can be read 16 bytes at a time
    return a.x_shared && a.vec_ok && a.gram != nullptr;
}

bool dense_window_wanted(const DenseArgs &a)
{
    if (!dense_window_supported(a)) return false;
    const int64_t path = a.tune->get(OCO_OPT_DENSE_PATH);
    if (path == 1) return a.d > 64 * kWave;                     // the register kernel cannot hold more
    if (path == 2) return true;
    // measured on MI355X: c4 (16384 learners, d = 4096) 58 ms against the register kernel's 138 ms; c3 (4352
    // learners, d = 1000) 50 ms against 62 ms.  Fewer learners stay with the register kernel (a round costs about
    // 0.35 us here whatever d is, as long as the workgroups fit the chip at once), and so do narrower models: from 3072
    // learners on this kernel would be up to twice as fast there (8192 learners, 2048 rounds 1.48 / 0.74 ms at d = 16, 1.65 / 1.02 at
    // d = 512), but its float32 hand-overs make the results less accurate against float64 (4096 learners, 1024 squared-loss
    // rounds of d = 256: iterates 4.5e-7 / 1.3e-6, combined 1.7e-7 / 7.4e-7) and dependent on how the horizon is cut.
    return a.d > 64 * kWave || ((int64_t)a.R * a.K >= 2048 && a.d >= 512);
}

namespace {

// Loading wavefronts: whether a call of nwin windows takes its products as bfloat16 parts or in float32.  Parts need iterates in
// blocks or at least whole 64-byte pieces for the streaming hint: of rows that do not end with a block of 16, calls of 4096
// rounds take 10.5 ms in float32 and 14.7 in parts (d = 3000), 14.9 / 25.2 (d = 4100), 8.2 / 11.6 (2052); rows longer than a tile's blocks hold
// lose too (d = 8192 27.3 / 29.9, d = 6144 20.5 / 21.9; 16384 learners).  A call pays once for turning the iterates and for two thirds of the
// windows per launch, and gains by the window: 23 us while every compute unit has a workgroup, d = 4096, and two to three times that
// for the workgroups of a last, partial turn (200 us per window in float32 however few they are, 127 to 165 in parts).  Turned
// iterates cost 11 such gains per 256 workgroups, launches the rest up to 20.  Measured, ms per call, float32 / parts:
//   16384 learners (256 workgroups), d = 4096   64 rounds 0.73 / 0.99   512 2.25 / 2.53   1024 3.91 / 3.92   1280 4.78 / 4.66   4096 14.3 / 12.5
//                                    d = 2048   64 rounds 0.34 / 0.50   512 1.16 / 1.35   1024 2.10 / 2.14   1280 2.58 / 2.58   4096 7.74 / 7.11
//   17408 learners (272),            d = 4096   64 rounds 1.00 / 1.18   320 2.65 / 2.68    512 3.86 / 3.57   1024 7.27 / 5.97   4096 27.1 / 20.8
//   24576 learners (384),            d = 4096   64 rounds 1.05 / 1.37   320 2.64 / 2.94    512 3.85 / 3.90   1024 7.12 / 6.50   4096 26.7 / 22.0
//   28672 learners (448),            d = 4096   64 rounds 1.07 / 1.51   512 3.88 / 4.24    640 4.75 / 4.96   1024 7.11 / 6.89   4096 26.7 / 23.0
//   65536 learners (1024),           d = 4096   64 rounds 1.84 / 2.89   768 10.8 / 11.1   1024 14.2 / 14.0   1280 17.3 / 16.7   4096 53.9 / 46.7
// The linear loss stays in float32.  Its losses are the predictions themselves, summed over the rounds, and the 16-bit instructions' sums
// lean to one side by a few 2^-26 of a prediction: 1536 optimistic rounds of d = 2048 had cumulative losses 2.2e-6 off by 2-norm in
// parts, 5.3e-7 in float32 (d = 4096 9.3e-7 and 2.2e-7).  With the other losses none is further off (squared 1.9e-8 and 1.9e-8, logistic
// 2.0e-10 and 2.0e-10), and the iterates are nearer with all three (squared 5.8e-7 and 6.0e-7, logistic 1.3e-7 and 2.0e-7).
bool parts_pay(int64_t nq, int d, int nwin, int ncu, int loss)
{
    if (loss == 0 || d % 16 != 0 || d > kBlocksMaxD) return false;
    const int64_t wgs = (nq + kQT * kM - 1) / (kQT * kM), rest = wgs % ncu;
    const int64_t gain = wgs / ncu + (rest == 0 ? 0 : 2 * rest <= ncu ? 3 : 2);
    return nwin * gain * ncu >= 20 * wgs;
}

}  // namespace

hipError_t launch_dense_window(const DenseArgs &a0, int loss, hipStream_t s, const PieceHook *hook)
{
    DenseArgs a = a0;
    if (a.n <= 0) return hipSuccess;
    if (!dense_window_supported(a)) return hipErrorInvalidValue;
    const WinPlanD plan{a.t0, a.n};
    const int nwin = plan.count();
    const int nblk = (a.d + 15) / 16;
    const Scratch sc = scratch_layout(a.n_max, a.d);
    float *gram = a.gram, *gxt = gram + sc.gram_floats, *xq = gxt + sc.gram_floats, *xu = xq + sc.tile_floats;
    float *misc = xu + sc.tile_floats;
    {
        ComparatorGemmArgs g{};
        g.x = a.x; g.u = a.u; g.seg_start = a.seg_start; g.S = a.S; g.Z = a.Z; g.zl = a.zl;
        g.d = a.d; g.K = a.K; g.R = a.R; g.t0 = a.t0; g.n = a.n; g.vec_ok = a.vec_ok;
        hipError_t e = launch_comparator_gemm(g, s);
        if (e != hipSuccess) return e;
    }
    if (a.optimistic) {
        // ||x_t||^2 and <x_{t-1}, x_t> of the call's rounds (the first against the row kept from the call before)
        hipError_t e = launch_hint_scalars(a, s);
        if (e != hipSuccess) return e;
    }
    // where the iterates live: OCO_OPT_WINDOW_RESIDENT 1 registers (d <= 4096), 0 streamed (two tiles per
    // workgroup), 2 streamed (one tile, sixteen wavefronts), 3 streamed with loading wavefronts (four tiles),
    // 4 registers, two tiles per workgroup (d <= 1024).
    // Unset: streamed, two tiles -- on c4 as fast as the registers (every round row a wavefront loads
    // serves two tiles), on c3 half as many workgroups --, two tiles in registers where they fit and the
    // wavefronts have several blocks each (c3: 41.8 against 46.4 ms), or, with at least four tiles per compute unit's
    // workgroup on every one of 256 compute units and wide rows, the loading wavefronts (ms against two tiles, 16384
    // learners: c4 57.3 / 72.0; 4096 rounds of d = 2048 7.2 / 7.8; 2048 of d = 8192 13.6 / 16.3; 512 of d = 4096 2.43 / 2.40, 64 1.00 / 0.92;
    // c3, bound by the dependent rounds, which that kernel does not overlap: 101 / 47.5).
    // (5, the kernel with split coordinates, which did not take the call: as unset)
    const int64_t ropt = a.tune->get(OCO_OPT_WINDOW_RESIDENT) == 5 ? -1 : a.tune->get(OCO_OPT_WINDOW_RESIDENT);
    const bool fits = a.d <= 16 * kNW8 * 32;
    const bool many = (int64_t)a.R * a.K >= 1024 * kM && nblk >= 128;
    const bool fits2 = a.d <= 16 * kNW8 * 8;
    int mode = (ropt == 1 && fits) ? 0 : ropt == 2 ? 2 : (ropt == 3 || (ropt < 0 && many)) ? 3
               : ((ropt == 4 || (ropt < 0 && nblk >= 32)) && fits2) ? 4 : 1;
    if (a.optimistic && mode != 3 && mode != 4) mode = 1;    // (the optimistic update: three of the kernels only)
    const bool resident = mode == 0 || mode == 4;
    int ncu = 256;
    {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            ncu <= 0)
            ncu = 256;
    }
    const bool parts = mode == 3 && parts_pay((int64_t)a.R * a.K, a.d, nwin, ncu, loss);
    if (a.tune->get(OCO_OPT_VERBOSE) == 1)
        fprintf(stderr, "dense plan: windowed contraction kernel, %d windows in pieces of %lld, %d tiles, iterates %s\n",
                nwin, (long long)sc.piece_windows, (a.R * a.K + kM - 1) / kM,
                mode == 4 ? "in registers, two tiles per workgroup" : resident ? "in registers" : mode == 1 ? "streamed from HBM, two tiles per workgroup"
                : parts ? "streamed from HBM, four tiles per workgroup, rows through LDS in bfloat16 parts"
                : mode == 3 ? "streamed from HBM, four tiles per workgroup, rows through LDS" : "streamed from HBM");
    WindowKernel kern = nullptr;
    int waves = 0, tiles = 1, lds_bytes = 0;
    switch (loss) {
        case 0: kern = pick_window_kernel<0>(nblk, mode, parts, a.optimistic != 0, &waves, &tiles, &lds_bytes); break;
        case 1: kern = pick_window_kernel<1>(nblk, mode, parts, a.optimistic != 0, &waves, &tiles, &lds_bytes); break;
        case 2: kern = pick_window_kernel<2>(nblk, mode, parts, a.optimistic != 0, &waves, &tiles, &lds_bytes); break;
        default: return hipErrorInvalidValue;
    }
    const int ntiles = (a.R * a.K + kM * tiles - 1) / (kM * tiles);   // workgroups
    // The caller's work on a piece's rounds (the meta kernel) goes beside the window kernel of the following
    // piece where that leaves a quarter of the compute units or more without a workgroup (c3: 136 of 256;
    // 46.7 -> 45.8 ms per step: the window kernel is slower beside it, 6.25 against 5.72 ms per launch.
    // Handed over only behind the following piece's pre-passes: 46.2 ms).
    const bool beside = hook && hook->fn && 4 * (int64_t)ntiles <= 3 * (int64_t)ncu;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       lds_bytes);
    if (e != hipSuccess) return e;
    // rows in parts are half as long again: two thirds of the windows in the same scratch
    const int pw = parts ? std::max(1, (int)sc.piece_windows * 2 / 3) : (int)sc.piece_windows;
    if (parts && (size_t)pw * nblk * 2 * kSplitFloats > 2 * sc.tile_floats) return hipErrorInvalidValue;
    const bool blocked = parts && (int64_t)a.R * a.K % kM == 0;
    auto turn_blocks = [&](bool to_rows) -> hipError_t {
        if (!blocked) return hipSuccess;
        if (to_rows) hipLaunchKernelGGL(tile_blocks_kernel<true>, dim3((unsigned)(a.R * a.K / kM)), dim3(1024), 0, s, a.V, a.d);
        else hipLaunchKernelGGL(tile_blocks_kernel<false>, dim3((unsigned)(a.R * a.K / kM)), dim3(1024), 0, s, a.V, a.d);
        return hipGetLastError();
    };
    e = turn_blocks(false);
    if (e != hipSuccess) return e;
    for (int w0 = 0; w0 < nwin; w0 += pw) {
        const int nw = std::min<int>(pw, nwin - w0);
        hipLaunchKernelGGL(dense_tile_kernel, dim3((unsigned)nblk, (unsigned)nw), dim3(64), 0, s, a.x, a.d, plan, w0, xq,
                           parts ? nullptr : xu, misc);
        hipLaunchKernelGGL(dense_gram_kernel, dim3((unsigned)nw), dim3(512), 0, s, xq, nblk, gram, gxt);
        if (parts) {                                             // (in the place of the float32 copies, which the Gram matrices are done with)
            xu = xq + (size_t)pw * nblk * kSplitFloats;
            hipLaunchKernelGGL(dense_tile_split_kernel, dim3((unsigned)nblk, (unsigned)nw), dim3(64), 0, s, a.x, a.d, plan, w0, xq, xu);
        }
        e = clock_begin(a.clock, s, parts ? "dense_window_parts_kernel" : mode == 3 ? "dense_window_shared_kernel" : "dense_window_kernel");
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)ntiles), dim3(waves * kWave), lds_bytes, s, a, gram,
                           mode == 3 && !blocked ? nullptr : gxt, xq, xu, misc, plan, w0, nw);
        e = hipGetLastError();
        if (e == hipSuccess) e = clock_end(a.clock, s);
        if (e == hipSuccess && beside) {
            const int off = plan.start(w0), end = plan.start(w0 + nw - 1) + plan.len(w0 + nw - 1);
            e = hook->fn(hook->ctx, off, end - off);
        }
        if (e != hipSuccess) return e;
    }
    e = turn_blocks(true);
    if (e != hipSuccess) return e;
    return a.optimistic ? launch_keep_last_row(a, s) : hipSuccess;
}

}  // namespace oco
