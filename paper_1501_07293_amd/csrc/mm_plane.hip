// mm_plane.hip -- y forward, z k-space and y inverse of one x bin in one work-group, the
// z lines in registers.
#include <algorithm>

#include "mm_rline.hpp"

namespace mm {

// One work-group per x bin holds the bin's 3 nz rows in LDS (only them: the padding planes
// never leave the registers).  The y lines run as in body_ryz; then a thread takes a whole
// column ky: the z lines of the three components, transformed, multiplied (Eq. 14) and
// transformed back in its registers, with no exchange and no barrier between; then the y
// lines back.  In place of three launches and five sweeps over a spectrum of Py rows a
// bin, the ny rows are read once and written once.
//
// What bounds it is the chain of one work-group (y stages, a column, y stages), a work-group
// a CU: so it pays on small planes, where the three launches are bound by theirs, and loses
// on large ones, whose launches are bound by memory (plane_threads).
constexpr int kPlaneMaxThreads = 512;
// LDS row: odd, and one entry longer than the line, which columns past the last work on
__host__ __device__ constexpr int plane_row(int Py) { return (Py + 1) | 1; }
static size_t plane_lds_bytes(int Py, int nz, size_t esz) { return (size_t)3 * nz * plane_row(Py) * 2 * esz; }

// One column: entry z of component c at q[c cs + z zs], z < nz.
template <typename T, int PZ>
__device__ __forceinline__ void plane_column(cpx<T>* q, int cs, int zs, int nz, Buf K, unsigned ko, unsigned kcs,
                                             unsigned kzs, T sy)
{
    constexpr int H = PZ / 2;
    cpx<T> v[3][PZ];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int z = 0; z < PZ; ++z) {
            v[c][z] = cpx<T>{(T)0, (T)0};
            if (z < nz) v[c][z] = q[c * cs + z * zs];
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) Dft<T, PZ>::run(v[c]);
#pragma unroll
    for (int kz = 0; kz <= H; ++kz) {
        T k[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) k[c] = buf_ld<T>(K, ko, (unsigned)c * kcs + (unsigned)kz * kzs);
        k[1] *= sy;  // mirrored ky: xy and yz odd in y
        k[4] *= sy;
        tensor_product(&v[0][kz], &v[1][kz], &v[2][kz], k);
        if (kz > 0 && 2 * kz < PZ) {  // mirrored kz: xz and yz odd in z
            k[2] = -k[2];
            k[4] = -k[4];
            tensor_product(&v[0][PZ - kz], &v[1][PZ - kz], &v[2][PZ - kz], k);
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        Dft<T, PZ>::run(v[c]);
#pragma unroll
        for (int z = 0; z < PZ; ++z)
            if (z < nz) q[c * cs + z * zs] = v[c][z];
    }
}

// The z lengths a kernel serves: up to 8 points (134 registers in FP32, 239 in FP64), or 9
// to 12 in FP32 (197).  Longer lines spill: 14 to 20 points in FP32 made an RK4 step of
// 100x100x10 179 us instead of 121, 9 to 12 in FP64 one of 40x20x6 97 instead of 79.
#define MM_PLANE_CASES(X) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(12)

template <typename T, int RM, int ZLO, int ZHI>
__global__ __launch_bounds__(kPlaneMaxThreads) void k_plane(RYzArgs a, LinePlan pl, int Pz)
{
    extern __shared__ __attribute__((aligned(16))) char plane_smem[];
    cpx<T>* lds = reinterpret_cast<cpx<T>*>(plane_smem);
    const LineRegs sy(pl);
    const int kx = xcd_tile(blockIdx.x, gridDim.x);
    const int Py = sy.P, LP = plane_row(Py), ny = a.ny, nz = a.nz;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    constexpr unsigned CS = sizeof(cpx<T>), TS = sizeof(T);
    const Buf g = buf_of((const cpx<T>*)a.buf + (int64_t)kx * a.Sy);
    const Buf K = buf_of((const T*)a.kern + kx * a.k_xs);
    // y lines: line q = c nz + z at LDS row q, yper of them a round
    const int yper = a.zper, lines = 3 * nz;
    for (int q0 = 0; q0 < lines; q0 += yper) {
        const LaneOf w = rline_lane(sy, min(yper, lines - q0));
        const int q = q0 + w.l, c = nz == 1 ? q : div_by(q, a.zmul), z = q - c * nz;
        const unsigned at = ((unsigned)c * (unsigned)a.comp_stride + (unsigned)z * (unsigned)a.zs) * CS;
        cpx<T>* ln = lds + q * LP;
        rline_fft<T, RM, false, true>(
            sy, (const cpx<T>*)a.twsy, ln, w.u, w.real,
            [&](int e) { return buf_ld<cpx<T>>(g, e < ny ? at + (unsigned)e * CS : kBufNone); },
            [&](int e, cpx<T> x) { ln[e] = x; });
    }
    __syncthreads();
    for (int y0 = 0; y0 < Py; y0 += NT) {
        const int col = min(y0 + t, Py);  // Py: the spare entry of the rows
        const bool mir = 2 * col > Py;
        const unsigned ko = (unsigned)(mir ? Py - col : col) * TS, kcs = (unsigned)a.k_cs * TS, kzs = (unsigned)a.k_zs * TS;
        const T sgn = mir ? (T)-1 : (T)1;
        switch (Pz) {
#define X(PZ)                                                                                                  \
    case PZ:                                                                                                   \
        if constexpr (PZ >= ZLO && PZ <= ZHI) plane_column<T, PZ>(lds + col, nz * LP, LP, nz, K, ko, kcs, kzs, sgn); \
        break;
            MM_PLANE_CASES(X)
#undef X
        default: break;
        }
    }
    __syncthreads();
    for (int q0 = 0; q0 < lines; q0 += yper) {
        const LaneOf w = rline_lane(sy, min(yper, lines - q0));
        const int q = q0 + w.l, c = nz == 1 ? q : div_by(q, a.zmul), z = q - c * nz;
        const unsigned at = ((unsigned)c * (unsigned)a.comp_stride + (unsigned)z * (unsigned)a.zs) * CS;
        cpx<T>* ln = lds + q * LP;
        rline_fft<T, RM, true, false>(
            sy, (const cpx<T>*)a.twsy, ln, w.u, w.real, [&](int e) { return ln[e]; },
            [&](int e, cpx<T> x) { buf_st(g, e < ny ? at + (unsigned)e * CS : kBufNone, conj(x)); });
    }
}

static bool plane_length(int Pz)
{
    switch (Pz) {
#define X(PZ) case PZ:
        MM_PLANE_CASES(X)
#undef X
        return true;
    default: return false;
    }
}

// Where the pass takes the place of the three.  Measured per RK4 step with graph replay,
// three passes (or body_ryz, where the plane is small enough for it) -> this one.  Up to 8
// points along z, by the 3 nz Py entries of a plane: 8x8x4 (192) FP32 43.8 -> 39.7 us, FP64
// 53.1 -> 44.7; 60x40x3 (720) 68.6 -> 61.1 and 80.1 -> 69.4; 256x64x3 (1152) 88.4 -> 70.9
// and 141.6 -> 92.7; 256x64x4 (1536) 87.1 -> 75.6 and 112.3 -> 104.3; 250x120x4 (2880)
// 132.1 -> 111.1 and 175.4 -> 139.4; from 3072 on it is even or loses: 256x128x4 (3072)
// 101.4 -> 101.7 and 138.8 -> 140.0, 100x200x4 (4800) 112.2 -> 117.5, 300x300x3 (5400)
// 212.6 -> 255.0.  In FP64 many bins lose earlier, by the entries of them all:
// 500x100x3 (0.9 M) 237.6 -> 204.1, but 512x128x3 (1.2 M) 197.6 -> 202.1 and 1000x64x4
// (1.5 M) 260.6 -> 269.8; in FP32 these gain still (1000x64x4 188.7 -> 170.3).  9 to 12
// points in FP32: 20x20x5 (600) 58.0 -> 54.4, 60x60x5 (1800) 79.3 -> 71.4, but 100x100x5
// (3000) 90.9 -> 95.6.
int plane_threads(const LinePlan& y, int Pz, int hx, int nz, size_t esz, int* yper)
{
    if (y.ns <= 0 || !plane_length(Pz) || y.TL > kPlaneMaxThreads || nz > Pz) return 0;
    if (esz == 8 && Pz > 8) return 0;
    const int64_t plane = 3 * (int64_t)nz * y.P;
    if (Pz <= 8 ? plane >= 3072 : plane > 2048) return 0;
    if (plane * hx > (esz == 8 ? (int64_t)1 << 20 : (int64_t)1 << 21)) return 0;
    // the rounds of y lines the threads make necessary, evenly filled; threads for the
    // columns too
    const int lines = 3 * nz, most = kPlaneMaxThreads / y.TL, rounds = (lines + most - 1) / most;
    *yper = (lines + rounds - 1) / rounds;
    const int nt = (*yper * y.TL + 63) / 64 * 64, cols = (y.P + 63) / 64 * 64;
    return std::min(kPlaneMaxThreads, std::max(nt, cols));
}

template <typename T>
hipError_t launch_plane(const RYzArgs& a, const LinePlan& y, int Pz, hipStream_t st)
{
    const size_t lds = plane_lds_bytes(y.P, a.nz, sizeof(T));  // under 3072 + 9 nz entries: 50 KB
    if (a.nt > kPlaneMaxThreads || a.zper * y.TL > a.nt || a.zper < 1 || a.nz > Pz || !plane_length(Pz) ||
        lds > 64 * 1024)
        return hipErrorInvalidValue;
    if (a.hx <= 0) return hipSuccess;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(a.hx), dim3(a.nt), lds, st, a, y, Pz);
        return hipGetLastError();
    };
    bool small = true;
    for (int q = 0; q < y.ns; ++q) small = small && y.R[q] <= 10;
    if (Pz <= 8) return small ? go(k_plane<T, 10, 3, 8>) : go(k_plane<T, 16, 3, 8>);
    if constexpr (sizeof(T) == 4) return small ? go(k_plane<T, 10, 9, 12>) : go(k_plane<T, 16, 9, 12>);
    return hipErrorInvalidValue;
}
template hipError_t launch_plane<float>(const RYzArgs&, const LinePlan&, int, hipStream_t);
template hipError_t launch_plane<double>(const RYzArgs&, const LinePlan&, int, hipStream_t);

}  // namespace mm
