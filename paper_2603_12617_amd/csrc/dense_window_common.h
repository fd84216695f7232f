// What the kernels that work a shared dense stream in windows of 64 rounds have in common: the plan of
// a call's windows, the layout of the tiled round rows, and the dependent rounds of a window.
#pragma once
#include "oco_internal.h"

#include <type_traits>
#include <utility>

namespace oco {
namespace {

constexpr int kB = 64;            // rounds per window
constexpr int kM = 16;            // learners per tile
constexpr int kGStride = 18;      // doubles per (round, quad lane) row of the masked Gram table (16 + padding, where quad lane 0's row keeps ||x||^2 as a float)
constexpr int64_t kPieceBytes = 64ll << 20;   // stream per launch (each tiled copy is as large)
constexpr int kTileFloats = kB * 16;          // one window x one block of 16 coordinates
// A little scratch that lets the streamed sweep load and store without branches (a load or store
// that may or may not have been issued makes every later wait a wait for everything): lanes
// without a learner or past d read kMiscZeros zero floats and write to a sink of their own.
constexpr int kMiscZeros = 16, kMiscFloats = kMiscZeros + 1024 * 4;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
static_assert(kGStride % 2 == 0, "rows of the Gram table start on 16 bytes");

struct WinPlanD {
    int64_t t0;      // absolute round of the call's first round
    int n;           // rounds in the call
    __host__ __device__ int first_len() const { const int f = (int)(kB - t0 % kB); return f < n ? f : n; }
    __host__ __device__ int count() const { const int f = first_len(); return 1 + (n - f + kB - 1) / kB; }
    __host__ __device__ int start(int w) const { return w == 0 ? 0 : first_len() + (w - 1) * kB; }
    __host__ __device__ int len(int w) const { const int s = start(w); const int l = w == 0 ? first_len() : kB; return l < n - s ? l : n - s; }
};

// every lane of a quad gets the value of the quad's lane SEL
template <int SEL> __device__ __forceinline__ double quad_bcast(double v)
{
    constexpr int ctrl = SEL * 0x55;                             // quad_perm [SEL, SEL, SEL, SEL]
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), ctrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose index is a
// compile-time constant in every iteration (register arrays indexed by it stay in registers)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// The 64 dependent rounds of window k for the tile's 16 learners: wavefront 0, lane = 4 learner
// + quad lane s; quad lane s carries the pending predictions of the rounds t2 = 4 j + s.
// In: q0 = W' X_k^T with W' the iterates before the step of window k - 1 (or the stored ones, for the
// launch's first window), pmul and corr such that pmul q0 + corr = W_k X_k^T; labels, G; n2 = ||w_k||^2.
// Out (LDS buffer k % 2): predictions, -Bm, F = fscale f_0 ... f_63; returns F; n2 becomes ||w_{k+1}||^2
// by the scalar identity, *projected whether any round of the window projected this learner.
// Straight-line code: a window shorter than 64 rounds (first / last window of a call) runs its
// missing rounds as rounds without a step (a = 0, so f = 1 and no pending prediction moves; their
// rows of G are zero).
// The scalars the optimistic update (Eq. (3)) carries from round to round: the hint is ha x_{t-1},
// hp = <w^_t, x_{t-1}>, x2p = ||x_{t-1}||^2 (the vector the sweeps move is then the intermediate model w^).
struct Hint { float ha, hp, x2p; };

template <int LOSS, class Lds, bool OPT = false>
__device__ __forceinline__ double chain_window(char *lds, int buf, int m, int lane, int wl, float eta, double D, double pmul,
                                               double fscale, double &n2, bool &projected, Hint *hint = nullptr)
{
    using GT = typename Lds::G;
    using ST = typename Lds::S;
    const int lc = lane >> 2, s = lane & 3;
    const GT *gd = reinterpret_cast<const GT *>(lds + Lds::gd) + s * kGStride;
    const float *x2d = reinterpret_cast<const float *>(reinterpret_cast<const GT *>(lds + Lds::gd) + 16);
    constexpr int kX2 = 4 * kGStride * (int)(sizeof(GT) / sizeof(float));   // floats from one round's ||x||^2 to the next
    const ST *q0d = reinterpret_cast<const ST *>(lds + Lds::q0 + m * Lds::tile_s) + s * kM + lc;
    const float *cr = reinterpret_cast<const float *>(lds + Lds::corr + m * Lds::tile_f) + s * kM + lc;
    ST *fl = reinterpret_cast<ST *>(lds + Lds::fl + m * Lds::tile_s) + lc;
    const float *yb = reinterpret_cast<const float *>(lds + Lds::yb + buf * Lds::yb_bytes + m * Lds::tile_f) + lc;
    float *zb = reinterpret_cast<float *>(lds + Lds::zb + buf * Lds::zb_bytes + m * Lds::tile_f) + lc;
    float *stl = reinterpret_cast<float *>(lds + Lds::st + m * Lds::tile_f) + lc;
    const float Df = (float)D, D2f = Df * Df;
    const float eta2 = 2.f * eta;
    bool anyp = false;

    double p[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
        p[j] = Lds::has_corr ? fma(pmul, (double)q0d[4 * j * kM], (double)cr[4 * j * kM]) : pmul * (double)q0d[4 * j * kM];

    // A round has a short dependent part (prediction -> slope -> step -> norm -> projection factor
    // -> next prediction) and a wide independent one (its update of the pending predictions).  The
    // dependent part runs in float32: the next prediction is taken from the float64 pending value
    // by one float32 step, f (p - a G), as exact as a float32 inner product of that size; the
    // squared norm is carried in float32 within the window like the register kernel carries it
    // between its exact measurements (the caller re-anchors it every window), or, with Lds::carry_norm, in float64 and
    // as the factor applied leaves it: taken as D^2 after a projection it loses the errors of the factors, which then
    // add up over the window (norm off by 1.5e-7 after 56 rounds, 9e-8 on the register kernel; so 2.8e-8).  The pending
    // predictions themselves stay float64 (their recurrence is 64 rounds long); round t - 1's
    // update of them shares a scheduling region with the dependent part of round t and fills its
    // latencies.
    double gahead[16];                // the coming round's row of G
    if constexpr (Lds::g_reads == 2) {
#pragma unroll
        for (int j = 0; j < 16; j += 2) {
            const d2 g2 = *reinterpret_cast<const d2 *>(gd + j);
            gahead[j] = g2[0];
            gahead[j + 1] = g2[1];
        }
    }
    double gprev[16];                 // round t - 1's row of G (elements j >= (t - 1) / 4)
    double aprev = 0.0, fprev = 1.0;
    float n2f = (float)n2;
    double n2c = n2;                  // ||w_t||^2 where Lds::carry_norm
    float znext = (float)p[0];        // this lane's candidate for the next prediction (round 0: lane 0's is the one)
    // label and ||x||^2 of a round are read from LDS one round ahead: they are the first things the
    // dependent part needs, and nothing else would cover the latency of the read
    float ynext = yb[0], x2next = x2d[0];
    const float *hg = reinterpret_cast<const float *>(lds + Lds::hg + buf * Lds::hg_bytes);
    float gnext = OPT ? hg[0] : 0.f;
    float ha = 0.f, hp = 0.f, x2p = 0.f;
    if (OPT) { ha = hint->ha; hp = hint->hp; x2p = hint->x2p; }
    static_for<kB>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        constexpr int j0 = t >> 2;                                   // pending elements of this lane: j >= j0
        constexpr int jn = (t + 1) >> 2;                             // holds the prediction of round t + 1
        // this round's row of G.  Two entries at a time from an even one on are 16-byte reads whose offset is a
        // constant (8-byte pairs reach 2 KB only: an address computed for each was one instruction in twelve of a
        // round); read a round ahead, nothing waits for them.  Which form a kernel takes is what its registers allow:
        // dense_window_kernel spills 130 more with the rows a round ahead, dense_window_shared_kernel is 0.6 % slower
        // with the 16-byte reads (piecewise streams of d = 1000 gain 1.5 % by them).
        constexpr int je = Lds::g_reads > 0 ? j0 & ~1 : j0;
        double gr[16 - je];
        if constexpr (Lds::g_reads == 2) {
#pragma unroll
            for (int j = je; j < 16; ++j) gr[j - je] = gahead[j];
            if constexpr (t + 1 < kB) {
#pragma unroll
                for (int j = jn & ~1; j < 16; j += 2) {
                    const d2 g2 = *reinterpret_cast<const d2 *>(gd + (t + 1) * 4 * kGStride + j);
                    gahead[j] = g2[0];
                    gahead[j + 1] = g2[1];
                }
            }
        } else if constexpr (Lds::g_reads == 1) {
#pragma unroll
            for (int j = je; j < 16; j += 2) {
                const d2 g2 = *reinterpret_cast<const d2 *>(gd + t * 4 * kGStride + j);
                gr[j - je] = g2[0];
                gr[j - je + 1] = g2[1];
            }
        } else {
#pragma unroll
            for (int j = j0; j < 16; ++j) gr[j - j0] = gd[t * 4 * kGStride + j];
        }
        const float yt = ynext, x2t = x2next, g01t = gnext;
        if constexpr (t + 1 < kB) {
            ynext = yb[(t + 1) * kM];
            x2next = x2d[(t + 1) * kX2];
            if (OPT) gnext = hg[t + 1];
        }
        if constexpr (t > 0) {
            constexpr int jp0 = (t - 1) >> 2;
#pragma unroll
            for (int j = jp0; j < 16; ++j) p[j] = fprev * fma(-aprev, gprev[j], p[j]);
        }
        const float z32 = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(znext), (t & 3) * 0x55, 0xF, 0xF, false));   // <w_t, x_t>
        // the prediction that is played and scored: plain, z32; optimistic, that of w_t = s (w^_t - ha x_{t-1})
        // with s from ||w^_t - ha x_{t-1}||^2, all from scalars (z32 is then <w^_t, x_t>)
        float zp = z32;
        if (OPT) {
            const float mf = fmaf(ha * ha, x2p, fmaf(-2.f * ha, hp, n2f));
            const float sp = mf > D2f ? Df * __builtin_amdgcn_rsqf(mf) : 1.f;
            zp = sp * fmaf(-ha, g01t, z32);
        }
        // a_t = eta c_t; for the squared loss eta * 2 (z - y) = (2 eta) (z - y) exactly
        float a32 = LOSS == 1 ? eta2 * (zp - yt) : eta * slope<LOSS>(zp, yt);
        a32 = t < wl ? a32 : 0.f;
        // ||w_t - a_t x_t||^2 and the projection factor
        const float dn = fmaf(a32, x2t, -2.f * z32);                 // (||w_t - a_t x_t||^2 - ||w_t||^2) / a_t
        double m2d = 0.0;
        float m2;
        if constexpr (Lds::carry_norm) { m2d = fmax(fma((double)a32, (double)dn, n2c), 0.0); m2 = (float)m2d; }
        else m2 = fmaxf(fmaf(a32, dn, n2f), 0.f);
        const bool pj = m2 > D2f;
        const float f32v = pj ? Df * __builtin_amdgcn_rsqf(m2) : 1.f;
        if constexpr (Lds::carry_norm) { n2c = m2d * (double)f32v * (double)f32v; n2f = (float)n2c; }
        else n2f = pj ? D2f : m2;
        anyp = anyp || pj;
        zb[t * kM] = zp;                                             // (the quad's four lanes write the same value)
        stl[t * kM] = a32;
        fl[t * kM] = (ST)f32v;
        if (OPT) {                                                   // next round's hint and <w^_{t+1}, x_t>
            const bool live = t < wl;                                // (selects, not a branch: the rounds stay straight-line code)
            hp = live ? f32v * fmaf(-a32, x2t, z32) : hp;
            ha = live ? a32 : ha;
            x2p = live ? x2t : x2p;
        }
        // (p[jn] has the updates of the rounds before this one: the loop above ran)
        if constexpr (jn < 16) znext = f32v * fmaf(-a32, (float)gr[jn - je], (float)p[jn]);
#pragma unroll
        for (int j = j0; j < 16; ++j) gprev[j] = gr[j - je];
        aprev = (double)a32;
        fprev = (double)f32v;
        __builtin_amdgcn_sched_barrier(0);                           // at most two rounds overlap: registers
    });
    n2 = Lds::carry_norm ? n2c : (double)n2f;
    if (OPT) { hint->ha = ha; hint->hp = hp; hint->x2p = x2p; }

    // Bm[r] = a_r f_r f_{r+1} ... f_63 and F = fscale f_0 ... f_63: quad lane s takes the rounds
    // 16 s .. 16 s + 15 backwards, then the quad's products are combined
    float *bm = reinterpret_cast<float *>(lds + Lds::bm + buf * Lds::bm_bytes + m * Lds::tile_f) + lc;
    float *fv = reinterpret_cast<float *>(lds + Lds::fv + buf * Lds::fv_bytes) + m * kM;
    double loc[16];
    double acc = 1.0;
#pragma unroll
    for (int k = 15; k >= 0; --k) {
        acc *= (double)fl[(16 * s + k) * kM];
        loc[k] = acc;
    }
    const double P0 = quad_bcast<0>(acc), P1 = quad_bcast<1>(acc), P2 = quad_bcast<2>(acc), P3 = quad_bcast<3>(acc);
    const double tail = s == 3 ? 1.0 : s == 2 ? P3 : s == 1 ? P2 * P3 : P1 * (P2 * P3);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int r = 16 * s + k;
        bm[r * kM] = -(float)((double)stl[r * kM] * (loc[k] * tail));
    }
    const double F = fscale * (P0 * (P1 * (P2 * P3)));
    if (s == 0) fv[lc] = (float)F;
    projected = anyp;
    return F;
}

}  // namespace

// scratch of the windowed kernels for calls of at most n_max rounds, in floats
size_t dense_window_scratch_floats(int64_t n_max, int64_t d);

}  // namespace oco
