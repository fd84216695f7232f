// The dependent rounds of a window (see dense_window_common.h), four learners to a wavefront.
#pragma once
#include "dense_window_common.h"

namespace oco {
namespace {

// every lane of a row of 16 gets the value of the row's lane SEL
template <int SEL> __device__ __forceinline__ double row_bcast(double v)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + SEL, 0xF, 0xF, false),
                            __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + SEL, 0xF, 0xF, false));
}
template <int SEL> __device__ __forceinline__ float row_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + SEL, 0xF, 0xF, true));
}

// sum over the lanes of a row of 16, the same in every lane (each step adds the sums of two halves of a coset)
__device__ __forceinline__ double row_sum(double v)
{
    static_for<4>([&](auto ic) __attribute__((always_inline)) {
        constexpr int ror = 0x120 + (8 >> decltype(ic)::value);     // row_ror 8, 4, 2, 1
        v += __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ror, 0xF, 0xF, false),
                              __builtin_amdgcn_mov_dpp(__double2loint(v), ror, 0xF, 0xF, false));
    });
    return v;
}

// What the dependent rounds of a window read of its rows alone, in LDS: G[t][t2] for t2 > t, else 0, and of every round
// ||x_t||^2 / 2 and <x_{t-1}, x_t> (optimistic update).  Lane s of the 16 lanes that share a learner reads the entries
// t2 = 16 j + s of a row, two j at a time.
constexpr int kL = 16, kNP = kB / kL;
constexpr int kGramBytes = kB * kB * 8, kScalBytes = kB * 2 * 8;
// Strides of a tile's arrays in LDS, such that the lanes of a learner and those of a row are in banks of their own: labels and
// predictions learner by learner, W X^T and what the rounds record (float64) and -Bm (float32) round by round.
constexpr int kYStride = 68, kQStride = 18, kBmStride = 20;
constexpr int kYBytes = kM * kYStride * 4, kQBytes = kB * kQStride * 8, kBmBytes = kB * kBmStride * 4;
// entry (t, t2) of the Gram matrix
__device__ __forceinline__ void put_gram(double *gd, double *scal, int t, int t2, double v)
{
    gd[((t * (kNP / 2) + (t2 / kL >> 1)) * kL + t2 % kL) * 2 + (t2 / kL & 1)] = t2 > t ? v : 0.0;
    if (t2 == t) scal[2 * t] = 0.5 * v;
}

// The 64 dependent rounds of window k for four learners of a tile of 16: one wavefront, 16 lanes per learner, lane s of them
// with the pending inner products of the rounds t2 = 16 j + s.  (Four wavefronts run a tile's rounds; `part` says which this is.)
// In: q0 such that pmul q0 = W_k X_k^T, labels, the tables above; n2 = ||w_k||^2.
// (tab: where the two tables lie, in bytes past Lds::gd and Lds::scal.)
// Out: predictions, -Bm, F = fscale times what is left of w_k in w_{k+1}; n2 becomes ||w_{k+1}||^2 by the scalar identity.
//
// Within the window an iterate is w_t = v_t / s_t, as in the register kernel: a step is linear in v,
//     v <- v - b x_t,   b = a_t s_t,   a_t = eta c_t,
// and a projection only raises s.  So a round touches a pending inner product once, p[t2] -= b G[t][t2] (no factor of the
// projection goes through the products, nor a scan of the factors through the window's steps afterwards: Bm[t] = b_t / s_end),
// and nothing of a round is a compare, a select or a branch: with h = ||v||^2 / 2,
//     h <- h + b (b ||x_t||^2 / 2 - p_t),   s <- max(s, sqrt(2 h) / D),
// the maximum of the norms so far, taken afresh from the norm whenever it acts, so that its rounding does not add up.  S below is
// s D / sqrt 2, hence S <- max(S, sqrt h); where a prediction is needed in the chain its reciprocal I <- min(I, rsq h) goes
// beside it.  All of it is float64, which a wavefront alone on its SIMD issues no slower than float32 (8 clocks for a
// multiply-add that waits for the one before, 5 for one that does not, 21 for a square root; measured) and which needs no
// conversions in between; v_sqrt_f64 and v_rsq_f64 are good to 5e-8, as good as their float32 forms.
// What bounds it: instructions.  A wavefront alone on its SIMD pays 7 clocks for each, whatever it waits for: 20 per round of the plain
// update with the squared loss (140 clocks), 42 of the optimistic one with the logistic loss (299); 128 / 140 / 217 clocks plain,
// 238 / 271 / 299 optimistic, linear / squared / logistic.  The quad of lanes per learner that chain_window gives a wavefront of
// sixteen learners takes 264 / 280 / 306 and 306 / 329 / 358: its lanes have sixteen pending products where these have four.
// s grows by the factor a step leaves the ball by, every round: every eighth round a learner whose s has grown beyond 2^20 is
// taken back to below 2 by a power of two (exact), so that the norm stays within float64 for steps up to 2^60 times the ball
// (chain_holds says for which configurations; others do not come here).
//
// Straight-line code: a window shorter than 64 rounds (first / last window of a call) runs its
// missing rounds with rows of G, labels and inner products of zero, which change nothing (the linear loss has a b there, which is
// left out of Bm).
template <int LOSS, class Lds, bool OPT>
__device__ __forceinline__ double chain_rounds(char *lds, int m, int part, int lane, int wl, float eta, double D, double pmul,
                                               double fscale, double &n2, Hint *hint, int tab = 0)
{
    constexpr bool RECIP = OPT || LOSS == 2;                     // the chain needs the predictions themselves
    constexpr int L = kL, NP = kNP;
    const int lc = part * (kWave / L) + lane / L, s = lane % L;
    const d2 *gd = reinterpret_cast<const d2 *>(lds + Lds::gd + tab) + s;
    const d2 *sc = reinterpret_cast<const d2 *>(lds + Lds::scal + tab);
    const double *q0d = reinterpret_cast<const double *>(lds + Lds::q0 + m * kQBytes) + s * kQStride + lc;
    double *rec = reinterpret_cast<double *>(lds + Lds::rec + m * kQBytes) + lc;          // b_t, or S_t where that gives all the rest
    const float *yb = reinterpret_cast<const float *>(lds + Lds::yb + m * kYBytes) + lc * kYStride;
    float *zb = reinterpret_cast<float *>(lds + Lds::zb + m * kYBytes) + lc * kYStride;
    const double kappa = 1.4142135623730951 / D, S0 = D * 0.70710678118654752;
    const float ikappa = (float)S0;
    const double e2 = 2.0 * (double)eta, ek = (double)eta * kappa, ey = -e2 * kappa;
    const double c1 = 1.4426950408889634 * S0;                   // exponent of the logistic slope, base 2

    double p[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) p[j] = pmul * q0d[L * j * kQStride];

    double h = 0.5 * n2, S = S0, I = kappa, A = 1.0;
    // optimistic update: the hint is u S x_{t-1} (u = kappa ha), hpv = <v_t, x_{t-1}>, x2p = ||x_{t-1}||^2 / 2
    double u = 0.0, hpv = 0.0, x2p = 0.0;
    if (OPT) { u = kappa * (double)hint->ha; hpv = (double)hint->hp; x2p = 0.5 * (double)hint->x2p; }
    // Label and row scalars of round 16 j + s, a lane each (from there to the row's lanes by one or two instructions, where an LDS
    // read costs 13 clocks): the label times -2 eta kappa for the squared loss, for the logistic one what its slope is of and is
    // multiplied with; ||x||^2 / 2, <x_{t-1}, x_t>.
    double ys[NP], xs[NP], gs[NP];
    float yc[NP], yk[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const float y = LOSS == 0 ? 0.f : yb[L * j + s];
        ys[j] = LOSS == 1 ? ey * (double)y : 0.0;
        yc[j] = LOSS == 2 ? (float)(c1 * (double)y) : 0.f;
        yk[j] = LOSS == 2 ? (float)(-ek * (double)y) : 0.f;
        xs[j] = sc[L * j + s][0];
        gs[j] = OPT ? sc[L * j + s][1] : 0.0;
    }
    int made = 0;                     // rounds whose prediction and b were made before the end (the same in every lane)
    // From what is recorded of this lane's round L j + s, S_t, and <v_t, x_t>, which the lane still holds: the prediction and b
    // (as in the chain, from the same numbers), b in the place of S_t.
    auto make_b = [&](int j) __attribute__((always_inline)) {
        const int t = L * j + s;
        const double St = rec[t * kQStride];
        zb[t] = (float)(p[j] * (__builtin_amdgcn_rcp(St) * S0));
        return LOSS == 1 ? fma(ys[j], St, e2 * p[j]) : ek * St;
    };
    d2 grow[NP / 2];                  // the row of G for the step that was just found, read a round before
    double pt, b;                     // <v_t, x_t> and b_t
    // Round t's prediction and step, from <v_t, x_t>, S, h and (optimistic update) the hint.  The inner product whose prediction
    // is played and scored: plain, pt; optimistic, that of r (v_t - u S x_{t-1}) with r from ||v_t - u S x_{t-1}||^2, all from scalars.
    auto find_b = [&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value, j = t / L, q = t % L;
        pt = row_bcast<q>(p[j]);                                     // <v_t, x_t>
        double w = pt, r = 1.0;
        if (OPT) {
            const double c = u * S;
            w = fma(-c, row_bcast<q>(gs[j]), pt);
            r = S * __builtin_amdgcn_rsq(fma(c, fma(c, x2p, -hpv), h));
   // (not a number, of a sum that rounds to below 0: taken as 1)
        }
        if (LOSS == 0) b = ek * S;
        if constexpr (RECIP) {
            const float wk = (float)(w * I);
            const float zk = OPT ? fminf((float)r, 1.f) * wk : wk;   // kappa times the prediction
            zb[t] = zk;                                         // (the lanes of a learner write the same value)
            if (LOSS == 2) {
                const float e = __builtin_amdgcn_exp2f(zk * row_bcast<q>(yc[j]));
                b = S * (double)(__builtin_amdgcn_rcpf(1.0f + e) * row_bcast<q>(yk[j]));
            }
        }
        if (LOSS == 1) {
            const double y = row_bcast<q>(ys[j]);
            b = OPT ? fma(fmin(r, 1.0), e2 * w, y * S) : fma(y, S, e2 * pt);
        }
        rec[t * kQStride] = RECIP ? b : S;
    };
#pragma unroll
    for (int i = 0; i < NP / 2; ++i) grow[i] = gd[i * L];
    find_b(std::integral_constant<int, 0>{});
    static_for<kB>([&](auto tc) __attribute__((always_inline)) {
        constexpr int t = decltype(tc)::value;
        constexpr int jn = (t + 1) / L;                              // holds the product of round t + 1
        __builtin_amdgcn_sched_barrier(0);
        // first what the next round waits for longest, and the reads for the one after
        d2 gr[NP / 2];
#pragma unroll
        for (int i = jn / 2; i < NP / 2; ++i) gr[i] = grow[i];
        if constexpr (jn < NP) p[jn] = fma(-b, gr[jn >> 1][jn & 1], p[jn]);
        const double x2 = row_bcast<t % L>(xs[t / L]);
        const double k = fma(b, x2, -pt);
        if (OPT) { u = b * I; hpv = -fma(b, x2, k); x2p = x2; }
        if constexpr (t + 1 < kB) {
            // (an entry that is not needed is not read either: its register would be taken again at once, and wait for the read)
            constexpr int jr = (t + 2) / L;
#pragma unroll
            for (int i = jr / 2; i < NP / 2; ++i) {
                const d2 *at = gd + ((t + 1) * (NP / 2) + i) * L;
                if (2 * i < jr) grow[i][1] = reinterpret_cast<const double *>(at)[1];
                else grow[i] = *at;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        h = fma(b, k, h);
        double root;                                                 // (not a number, of an h that rounds to below 0, or to it: S and I stay)
        if (RECIP) {
            const double ir = __builtin_amdgcn_rsq(h);
            root = h * ir;
            I = fmin(I, ir);
        } else {
            root = __builtin_amdgcn_sqrt(h);
        }
#pragma unroll
        for (int j = jn + 1; j < NP; ++j) p[j] = fma(-b, gr[j >> 1][j & 1], p[j]);
        S = fmax(S, root);
        if constexpr (t % 8 == 7 && t + 1 < kB) {
            const bool far = S > 0x1p20 * S0;
            if (__builtin_amdgcn_ballot_w64(far) != 0) {
                // a power of two off v: the pending products, the norm, what is recorded, and what is left of w_k
                const double f = far ? __builtin_amdgcn_ldexp(1.0, 1 - __builtin_amdgcn_frexp_exp(S * kappa)) : 1.0;
                if constexpr (!RECIP) {                              // (predictions first: S_t may vanish)
#pragma unroll
                    for (int j = 0; j <= t / L; ++j)
                        if (L * j + s >= made && L * j + s <= t) rec[(L * j + s) * kQStride] = make_b(j);
                    made = t + 1;
                }
#pragma unroll
                for (int j = 0; j < NP; ++j) p[j] *= f;
                h *= f * f;
                S *= f;
                A *= f;
                if (RECIP) I /= f;
                if (OPT) hpv *= f;
                for (int i = s; i <= t; i += L) rec[i * kQStride] *= f;
            }
        }
        if constexpr (t + 1 < kB) {
            find_b(std::integral_constant<int, t + 1>{});
        }
    });
    // W <- F W - Bm X_k
    const double left = 1.0 / (S * kappa);
    n2 = 2.0 * h * left * left;
    float *bm = reinterpret_cast<float *>(lds + Lds::bm + m * kBmBytes) + lc;
    float *fv = reinterpret_cast<float *>(lds + Lds::fv) + m * kM;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int t = L * j + s;
        double b;
        if (RECIP || t < made) b = rec[t * kQStride];
        else b = make_b(j);
        bm[t * kBmStride] = t < wl ? -(float)(b * left) : 0.f;
        if (RECIP) zb[t] *= ikappa;
    }
    if (OPT) {
        // the hint for the next window: the last round's step, from its prediction, and <w^, x> of its row
        const int te = wl - 1;
        double pe = 0.0;
#pragma unroll
        for (int j = 0; j < NP; ++j) pe = te / L == j ? p[j] : pe;
        pe = __shfl(pe, (lane & ~(L - 1)) | (te % L));
        const double x2e = sc[te][0];
        const float ze = zb[te], ye = yb[te];
        hint->ha = LOSS == 1 ? 2.f * eta * (ze - ye) : eta * slope<LOSS>(ze, ye);
        hint->hp = (float)(fma(-2.0 * rec[te * kQStride], x2e, pe) * left);
        hint->x2p = (float)(2.0 * x2e);
    }
    const double F = fscale * (A * left);
    if (s == 0) fv[lc] = (float)F;
    return F;
}

}  // namespace
}  // namespace oco
