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
bool dense_short_supported(const DenseArgs &a)
{
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
