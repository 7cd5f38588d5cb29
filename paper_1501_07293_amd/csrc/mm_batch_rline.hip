// mm_batch_rline.hip -- the batched form of the runtime-length register passes: one
// launch per pass over all grids that take it (a grid that does not has no tiles in the
// pass's prefix sums); bodies in mm_rline.hpp.
#include "mm_rline.hpp"

namespace mm {

extern __shared__ __align__(16) char batch_smem[];

template <typename T, bool INV>
__global__ __launch_bounds__(kBatchNT) void kbr_x(BatchPass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.n, tile);
    const BatchDesc& d = p.d[s];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(batch_smem);
    const cpx<T>* tws = p.tw + d.twx + d.Px;
    if constexpr (INV) {
        const RXArgs a{p.S + d.soff, p.out + d.moff, 3 * d.nz, d.ny, d.nx, d.Sy, tws, d.rs.lsh_i};
        body_rxinv<T, 16>(a, d.lx, tile - p.prefix[s], lds);
    } else {
        const RXArgs a{p.in + d.moff, p.S + d.soff, 3 * d.nz, d.ny, d.nx, d.Sy, tws, d.rs.lsh_f};
        body_rxfwd<T, 16>(a, d.lx, tile - p.prefix[s], lds);
    }
}

template <typename T, bool INV>
__global__ __launch_bounds__(kBatchNT) void kbr_y(BatchPass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.n, tile);
    const BatchDesc& d = p.d[s];
    const RYArgs a{p.S + d.soff, 3 * d.nz * d.hx, d.Sy, INV ? d.Py : d.ny, INV ? d.ny : d.Py,
                   p.tw + d.twy + d.Py, 0, d.rs.y};
    body_ryline<T, 16, INV>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T>
__global__ __launch_bounds__(kBatchNT) void kbr_kz(BatchPass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.n, tile);
    const BatchDesc& d = p.d[s];
    const int64_t plane = (int64_t)d.hx * d.Py;
    const RKzArgs a{p.S + d.soff, d.nz * plane, (int)plane, d.nz, d.Py, p.tw + d.twz + d.Pz, p.kern + d.koff,
                    d.oct, (int64_t)d.hx * (d.Py / 2 + 1), d.Py / 2 + 1, d.rs.csh};
    body_rkz<T, 16>(a, d.lz, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T>
__global__ __launch_bounds__(kBatchNT) void kbr_ky(BatchPass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.n, tile);
    const BatchDesc& d = p.d[s];
    const RKyArgs a{p.S + d.soff, (int64_t)d.hx * d.ny, d.ny, d.hx, d.ny, p.tw + d.twy + d.Py, p.kern + d.koff,
                    d.oct, d.Py / 2 + 1, d.rs.ky, d.pymul};
    body_rky<T, 16>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T>
__global__ __launch_bounds__(kBatchNT) void kbr_ky2(BatchPass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.n, tile);
    const BatchDesc& d = p.d[s];
    const int64_t plane = (int64_t)d.hx * d.ny;
    const RKy2Args a{p.S + d.soff, 2 * plane, plane, d.ny, d.hx, d.ny, p.tw + d.twy + d.Py, p.kern + d.koff,
                     d.oct, d.Py / 2 + 1, d.rs.ky2, d.pymul};
    body_rky2<T, 16>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T>
hipError_t launch_batch_rline(int which, const BatchPass<T>& p, int total_tiles, int inverse, size_t lds,
                              hipStream_t s)
{
    if (total_tiles <= 0) return hipSuccess;
    const dim3 grid(total_tiles), block(kBatchNT);
    switch (which) {
    case 0: hipLaunchKernelGGL((kbr_x<T, false>), grid, block, lds, s, p); break;
    case 1:
        if (inverse)
            hipLaunchKernelGGL((kbr_y<T, true>), grid, block, lds, s, p);
        else
            hipLaunchKernelGGL((kbr_y<T, false>), grid, block, lds, s, p);
        break;
    case 2: hipLaunchKernelGGL(kbr_kz<T>, grid, block, lds, s, p); break;
    case 3: hipLaunchKernelGGL((kbr_x<T, true>), grid, block, lds, s, p); break;
    case 4: hipLaunchKernelGGL(kbr_ky<T>, grid, block, lds, s, p); break;
    default: hipLaunchKernelGGL(kbr_ky2<T>, grid, block, lds, s, p); break;
    }
    return hipGetLastError();
}
template hipError_t launch_batch_rline<float>(int, const BatchPass<float>&, int, int, size_t, hipStream_t);
template hipError_t launch_batch_rline<double>(int, const BatchPass<double>&, int, int, size_t, hipStream_t);

}  // namespace mm
