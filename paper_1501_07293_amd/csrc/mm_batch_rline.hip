// mm_batch_rline.hip -- the batched form of the runtime-length register passes: one
// launch per pass over all grids that take it (a grid that does not has no tiles in the
// pass's prefix sums) and a range of radices; bodies in mm_rline.hpp.  512 grids of 32 to 128
// cells a side, 1 or 2 thick, FP32: 7.8 ms an RK4 step through the LDS-staged passes, 2.0 now.
// The instructions of the butterflies bound it; 512 threads a work-group only for the y
// k-space lines that 256 cannot hold (batch_shapes).
#include "mm_rline.hpp"

namespace mm {

extern __shared__ __align__(16) char batch_smem[];

template <typename T, int RM, bool INV>
__global__ __launch_bounds__(2 * kBatchNT) void kbr_x(BatchClass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.nmem, tile);
    const BatchDesc& d = p.d[p.members[s]];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(batch_smem);
    const cpx<T>* tws = p.tw + d.twx + d.Px;
    if constexpr (INV) {
        const RXArgs a{p.S + d.soff, p.out + d.moff, 3 * d.nz, d.ny, d.nx, d.Sy, tws, d.rs.lsh_i};
        body_rxinv<T, RM>(a, d.lx, tile - p.prefix[s], lds);
    } else {
        const RXArgs a{p.in + d.moff, p.S + d.soff, 3 * d.nz, d.ny, d.nx, d.Sy, tws, d.rs.lsh_f};
        body_rxfwd<T, RM>(a, d.lx, tile - p.prefix[s], lds);
    }
}

template <typename T, int RM, bool INV>
__global__ __launch_bounds__(2 * kBatchNT) void kbr_y(BatchClass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.nmem, tile);
    const BatchDesc& d = p.d[p.members[s]];
    const RYArgs a{p.S + d.soff, 3 * d.nz * d.hx, d.Sy, INV ? d.Py : d.ny, INV ? d.ny : d.Py,
                   p.tw + d.twy + d.Py, 0, d.rs.y};
    body_ryline<T, RM, INV>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T, int RM>
__global__ __launch_bounds__(2 * kBatchNT) void kbr_kz(BatchClass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.nmem, tile);
    const BatchDesc& d = p.d[p.members[s]];
    const int64_t plane = (int64_t)d.hx * d.Py;
    const RKzArgs a{p.S + d.soff, d.nz * plane, (int)plane, d.nz, d.Py, p.tw + d.twz + d.Pz, p.kern + d.koff,
                    d.oct, (int64_t)d.hx * (d.Py / 2 + 1), d.Py / 2 + 1, d.rs.csh};
    body_rkz<T, RM>(a, d.lz, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T, int RM>
__global__ __launch_bounds__(2 * kBatchNT) void kbr_ky(BatchClass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.nmem, tile);
    const BatchDesc& d = p.d[p.members[s]];
    const RKyArgs a{p.S + d.soff, (int64_t)d.hx * d.ny, d.ny, d.hx, d.ny, p.tw + d.twy + d.Py, p.kern + d.koff,
                    d.oct, d.Py / 2 + 1, d.rs.ky, d.pymul};
    body_rky<T, RM>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T, int RM>
__global__ __launch_bounds__(2 * kBatchNT) void kbr_ky2(BatchClass<T> p)
{
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int s = find_sample(p.prefix, p.nmem, tile);
    const BatchDesc& d = p.d[p.members[s]];
    const int64_t plane = (int64_t)d.hx * d.ny;
    const RKy2Args a{p.S + d.soff, 2 * plane, plane, d.ny, d.hx, d.ny, p.tw + d.twy + d.Py, p.kern + d.koff,
                     d.oct, d.Py / 2 + 1, d.rs.ky2, d.pymul};
    body_rky2<T, RM>(a, d.ly, tile - p.prefix[s], reinterpret_cast<cpx<T>*>(batch_smem));
}

template <typename T, int RM>
static hipError_t batch_rline_go(int pass, int nt, const BatchClass<T>& c, int tiles, int inverse, size_t lds,
                                 hipStream_t s)
{
    const dim3 grid(tiles), block(nt);
    switch (pass) {
    case kRPassX:
        if (inverse)
            hipLaunchKernelGGL((kbr_x<T, RM, true>), grid, block, lds, s, c);
        else
            hipLaunchKernelGGL((kbr_x<T, RM, false>), grid, block, lds, s, c);
        break;
    case kRPassY:
        if (inverse)
            hipLaunchKernelGGL((kbr_y<T, RM, true>), grid, block, lds, s, c);
        else
            hipLaunchKernelGGL((kbr_y<T, RM, false>), grid, block, lds, s, c);
        break;
    case kRPassKz: hipLaunchKernelGGL((kbr_kz<T, RM>), grid, block, lds, s, c); break;
    case kRPassKy: hipLaunchKernelGGL((kbr_ky<T, RM>), grid, block, lds, s, c); break;
    default: hipLaunchKernelGGL((kbr_ky2<T, RM>), grid, block, lds, s, c); break;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_batch_rline(int pass, int rmax, int nt, const BatchClass<T>& c, int tiles, int inverse,
                              size_t lds, hipStream_t s)
{
    if (nt != kBatchNT && nt != 2 * kBatchNT) return hipErrorInvalidValue;
    if (tiles <= 0) return hipSuccess;
    return rmax <= 10 ? batch_rline_go<T, 10>(pass, nt, c, tiles, inverse, lds, s)
                      : batch_rline_go<T, 16>(pass, nt, c, tiles, inverse, lds, s);
}
template hipError_t launch_batch_rline<float>(int, int, int, const BatchClass<float>&, int, int, size_t, hipStream_t);
template hipError_t launch_batch_rline<double>(int, int, int, const BatchClass<double>&, int, int, size_t, hipStream_t);

}  // namespace mm
