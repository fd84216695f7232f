// Short dense calls: the register kernel with everything around its rounds inside it, one kernel per call.
#include "dense_rounds_kernel.h"

#include <algorithm>

namespace oco {
namespace {

template <int NPL> hipError_t launch_npl(const DenseArgs &a, int loss, hipStream_t s)
{
    void (*kern)(const DenseArgs) = nullptr;
    switch (loss * 2 + (a.optimistic ? 1 : 0)) {
        case 0: kern = dense_rounds_kernel<NPL, 0, false, true>; break;
        case 1: kern = dense_rounds_kernel<NPL, 0, true, true>; break;
        case 2: kern = dense_rounds_kernel<NPL, 1, false, true>; break;
        case 3: kern = dense_rounds_kernel<NPL, 1, true, true>; break;
        case 4: kern = dense_rounds_kernel<NPL, 2, false, true>; break;
        case 5: kern = dense_rounds_kernel<NPL, 2, true, true>; break;
        default: return hipErrorInvalidValue;
    }
    // the ring is at least 24 KB: the meta work's 12.3 KB (K = 15) fit its space
    const size_t smem = sizeof(float) * ((size_t)kRing * a.rt * NPL * kWave + kWholeFloats);
    if (smem > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
    }
    hipError_t e = clock_begin(a.clock, s, "dense_round_kernel");
    if (e != hipSuccess) return e;
    const dim3 grid = a.x_shared ? dim3((unsigned)a.R, 1, 1) : dim3(1, (unsigned)a.R, 1);
    hipLaunchKernelGGL(kern, grid, dim3(DenseCfg<NPL>::MAXW * kWave), smem, s, a);
    e = hipGetLastError();
    return e != hipSuccess ? e : clock_end(a.clock, s);
}

int max_waves(int d)
{
    const int npl = (d + kWave - 1) / kWave;
    return npl <= 16 ? DenseCfg<16>::MAXW : npl <= 32 ? DenseCfg<32>::MAXW : DenseCfg<64>::MAXW;
}
static_assert(DenseCfg<1>::MAXW == DenseCfg<16>::MAXW && DenseCfg<2>::MAXW == DenseCfg<16>::MAXW &&
              DenseCfg<4>::MAXW == DenseCfg<16>::MAXW && DenseCfg<8>::MAXW == DenseCfg<16>::MAXW, "max_waves");

}  // namespace

// a.per_run = K + 1 wavefronts in one workgroup, a round per lane; a shared stream of several optimistic runs
// is left out (its workgroups all read the last row of the call before, which one of them would replace).
//
// A workgroup has all its wavefronts (max_waves) however few the run's tasks are, and beyond 1024 coordinates their registers
// let a compute unit hold one workgroup: more runs than compute units are then two turns, where the separate kernels pack the
// learners of a shared stream into fewer workgroups, or two workgroups of 1024 < d <= 2048 into a compute unit.  There the
// launches saved pay only for short calls.  16 calls, ms, separate kernels / one: shared streams, 512 runs of 1, d = 4096 1.10 /
// 1.19 (16 rounds), 1.34 / 1.63 (32), 1.80 / 2.50 (64), but 1.00 / 0.97 (8); d = 2048 0.98 / 0.84 (32), 1.26 / 1.36 (64); streams of
// their own, 341 runs of 2, 64 rounds, d = 1500 1.92 / 2.07, d = 2048 2.29 / 2.47, d = 4096 4.32 / 4.04; either, 64 rounds, 400 runs of 1,
// d = 700 0.99 / 0.93, 1.42 / 1.21.  Up to 256 runs the one kernel took less in every case tried (K = 1 ... 11, d = 10 ... 4096,
// 1 ... 64 rounds): 256 runs of 1, d = 4096, 64 rounds 1.72 / 1.28; 128 of 7 1.83 / 1.66; 256 of 2, d = 1000, 8 rounds 0.85 / 0.25.
bool dense_short_supported(const DenseArgs &a)
{
    constexpr int kComputeUnits = 256;
    if (a.R > kComputeUnits && a.d > 1024 && a.n > (a.d <= 2048 ? 32 : a.x_shared ? 8 : kWholeRounds)) return false;
    return a.n <= kWholeRounds && a.per_run <= max_waves(a.d) && !(a.optimistic && a.x_shared && a.R > 1);
}

hipError_t launch_dense_short(const DenseArgs &a, int loss, hipStream_t s)
{
    const int npl = (a.d + kWave - 1) / kWave;
    if (npl <= 1) return launch_npl<1>(a, loss, s);
    if (npl <= 2) return launch_npl<2>(a, loss, s);
    if (npl <= 4) return launch_npl<4>(a, loss, s);
    if (npl <= 8) return launch_npl<8>(a, loss, s);
    if (npl <= 16) return launch_npl<16>(a, loss, s);
    if (npl <= 32) return launch_npl<32>(a, loss, s);
    return launch_npl<64>(a, loss, s);
}

}  // namespace oco
