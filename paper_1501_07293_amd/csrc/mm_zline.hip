// mm_zline.hip -- the register z k-space pass (body_kspace_z) at lengths other than powers
// of two: the default padding of most layer counts.
//
// One thread holds a whole z line of one component, as in the power-of-two pass; the
// runtime-length pass (mm_rline.hpp) exchanges its stages through LDS and holds a radix's
// worth of registers for every length it serves.  Memory and its own butterflies bound it alike.
// It is the faster at every length below, in both precisions, also where FP64 lines take 244
// registers.  us a launch, that pass -> this one, FP32 and FP64: 200x150 cells a plane, 3 points
// 7.1 -> 6.8 and 9.6 -> 7.8, 12 points 10.5 -> 9.4 and 16.3 -> 13.0, 15 points 11.8 -> 11.4 and
// 19.9 -> 16.0, 30 points 31.3 -> 17.4 and 66.5 -> 28.2; 400x380: 7 points 19.5 -> 15.8 and 28.8 ->
// 27.1, 20 points 64.2 -> 33.2 and 142.1 -> 77.8, 30 points 122 -> 50.1 and 341 -> 116.
#include "mm_fast.hpp"

namespace mm {

template <typename T, int PZ>
__global__ __launch_bounds__(3 * kspace_z_cols<T>()) void k_kspace_z_mixed(KzArgs a)
{
    __shared__ cpx<T> sh[kspace_z_lds_elems<T, PZ>()];
    body_kspace_z<T, PZ>(a, xcd_tile(blockIdx.x, gridDim.x), sh);
}

template <typename T>
bool launch_kspace_z_mixed(const KzArgs& a, int PZ, hipStream_t s)
{
    constexpr int ZC = kspace_z_cols<T>();
    const int grid = (a.ncols + ZC - 1) / ZC;
    if (3 * a.comp_stride > INT32_MAX || 6 * a.k_cs > INT32_MAX) return false;  // 32-bit offsets
    if (grid <= 0) return true;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(3 * ZC), 0, s, a);
        return true;
    };
    switch (PZ) {
    case 3: return go(k_kspace_z_mixed<T, 3>);
    case 5: return go(k_kspace_z_mixed<T, 5>);
    case 6: return go(k_kspace_z_mixed<T, 6>);
    case 7: return go(k_kspace_z_mixed<T, 7>);
    case 9: return go(k_kspace_z_mixed<T, 9>);
    case 10: return go(k_kspace_z_mixed<T, 10>);
    case 12: return go(k_kspace_z_mixed<T, 12>);
    case 14: return go(k_kspace_z_mixed<T, 14>);
    case 15: return go(k_kspace_z_mixed<T, 15>);
    case 18: return go(k_kspace_z_mixed<T, 18>);
    case 20: return go(k_kspace_z_mixed<T, 20>);
    case 21: return go(k_kspace_z_mixed<T, 21>);
    case 24: return go(k_kspace_z_mixed<T, 24>);
    case 25: return go(k_kspace_z_mixed<T, 25>);
    case 28: return go(k_kspace_z_mixed<T, 28>);
    case 30: return go(k_kspace_z_mixed<T, 30>);
    default: return false;
    }
}

template bool launch_kspace_z_mixed<float>(const KzArgs&, int, hipStream_t);
template bool launch_kspace_z_mixed<double>(const KzArgs&, int, hipStream_t);

}  // namespace mm
