// mm_rfused.hip -- kernels of the fused stage pass and the fused adjoint stage for x
// lengths without a size-specialised pass (bodies in mm_rfused.hpp).
#include <algorithm>

#include "mm_rfused.hpp"

namespace mm {

constexpr int kRfMaxThreads = 512;
constexpr size_t kRfLds = 64 * 1024;
constexpr int kRfPrefetchGroups = 256;  // as the size-specialised form (mm_fused.hip)

extern __shared__ __align__(16) char rfused_smem[];

template <typename T, int RM, int PRE>
__global__ __launch_bounds__(kRfMaxThreads) void k_rfused_stage(FusedStageArgs<T> f, RFusedArgs g, LinePlan s)
{
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(rfused_smem);
    T* cell = reinterpret_cast<T*>(lds + 3 * rfused_region(g.L, s.P));
    body_rfused_stage<T, RM, PRE>(f, g, s, xcd_tile(blockIdx.x, gridDim.x), lds, cell);
}

template <typename T, int RM>
__global__ __launch_bounds__(kRfMaxThreads) void k_rfused_adjoint(FusedAdjArgs<T> f, RFusedArgs g, LinePlan s)
{
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(rfused_smem);
    T* cell = reinterpret_cast<T*>(lds + 3 * rfused_region(g.L, s.P));
    body_rfused_adjoint<T, RM>(f, g, s, xcd_tile(blockIdx.x, gridDim.x), lds, cell);
}

static size_t rfused_lds(int L, int P, int nx, size_t esz)
{
    return (size_t)3 * rfused_region(L, P) * 2 * esz + (size_t)3 * 2 * L * (nx + 1) * esz;
}
static int rfused_threads(int L, const LinePlan& s) { return std::max(256, (3 * L * s.TL + 63) / 64 * 64); }

int rfused_lines(const LinePlan& s, int nx, int rows, size_t esz)
{
    if (s.ns == 0) return 0;
    for (int L = rows >= 2048 ? 4 : (rows >= 1024 ? 2 : 1); L >= 1; L /= 2)
        if (rfused_threads(L, s) <= kRfMaxThreads && rfused_lds(L, s.P, nx, esz) <= kRfLds) return L;
    return 0;
}

// the arguments every form shares; false where the work-group does not fit
static bool rfused_args(RFusedArgs* g, const LinePlan& s, const void* S_in, void* S_out, int64_t sy, const void* tws,
                        int nx, int ny, int nz, int L, size_t esz, int* grid, int* nt, size_t* lds)
{
    *g = RFusedArgs{S_in, S_out, sy, tws, nx, ny, nz, L, L == 4 ? 3 : (L == 2 ? 2 : 1), div_mul(s.P / 2 + 1)};
    *grid = nz * ((ny + 2 * L - 1) / (2 * L));
    *nt = rfused_threads(L, s);
    // a work-group a CU or fewer: a thread a cell, up to 512.  RK4 step, FP32: 150x100x1 70.1 ->
    // 65.7 us, 250x60x2 82.9 -> 78.6, 200x100x4 98.1 -> 95.0; FP64 loses (200x40x1 72.9 -> 78.7,
    // 200x100x4 119.3 -> 122.4)
    if (esz == 4 && *grid <= kRfPrefetchGroups) *nt = std::max(*nt, std::min(kRfMaxThreads, (2 * L * nx + 63) / 64 * 64));
    *lds = rfused_lds(L, s.P, nx, esz);
    return s.ns > 0 && (L == 1 || L == 2 || L == 4) && *nt <= kRfMaxThreads && *lds <= kRfLds;
}

static bool small_radices(const LinePlan& s)
{
    for (int q = 0; q < s.ns; ++q)
        if (s.R[q] > 10) return false;
    return true;
}

template <typename T>
bool launch_rfused_stage(const FusedStageArgs<T>& f, const void* tws, const LinePlan& s, int L, hipStream_t st)
{
    RFusedArgs g;
    int grid, nt;
    size_t lds;
    if (f.g.per != 0 || !rfused_args(&g, s, f.S_in, f.S_out, f.sy, tws, f.g.nx, f.g.ny, f.g.nz, L, sizeof(T), &grid,
                                     &nt, &lds))
        return false;
    if (grid <= 0) return true;
    // cells per thread whose loads go out with the gather's
    const int nc = (2 * L * f.g.nx + nt - 1) / nt, pre = grid <= kRfPrefetchGroups && nc <= 2 ? nc : 0;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lds, st, f, g, s);
        return true;
    };
    if (small_radices(s))
        return pre == 1 ? go(k_rfused_stage<T, 10, 1>)
                        : (pre == 2 ? go(k_rfused_stage<T, 10, 2>) : go(k_rfused_stage<T, 10, 0>));
    return pre == 1 ? go(k_rfused_stage<T, 16, 1>)
                    : (pre == 2 ? go(k_rfused_stage<T, 16, 2>) : go(k_rfused_stage<T, 16, 0>));
}

template <typename T>
bool launch_rfused_adjoint(const FusedAdjArgs<T>& f, const void* tws, const LinePlan& s, int L, hipStream_t st)
{
    RFusedArgs g;
    int grid, nt;
    size_t lds;
    if (f.a.per != 0 || !rfused_args(&g, s, f.S_in, f.S_out, f.sy, tws, f.a.nx, f.a.ny, f.a.nz, L, sizeof(T), &grid,
                                     &nt, &lds))
        return false;
    if (grid <= 0) return true;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), lds, st, f, g, s);
        return true;
    };
    return small_radices(s) ? go(k_rfused_adjoint<T, 10>) : go(k_rfused_adjoint<T, 16>);
}

template bool launch_rfused_stage<float>(const FusedStageArgs<float>&, const void*, const LinePlan&, int, hipStream_t);
template bool launch_rfused_stage<double>(const FusedStageArgs<double>&, const void*, const LinePlan&, int, hipStream_t);
template bool launch_rfused_adjoint<float>(const FusedAdjArgs<float>&, const void*, const LinePlan&, int, hipStream_t);
template bool launch_rfused_adjoint<double>(const FusedAdjArgs<double>&, const void*, const LinePlan&, int, hipStream_t);

}  // namespace mm
