// mm_tiny.hip -- RK4 steps of a grid so small that one work-group holds all of it: every
// stage of every step of a call in one launch.
//
// Two launches a stage (the y k-space pass and the fused stage pass) take 3.7 to 4 us each
// on such a grid, most of it the way to memory and back and the gap between launches. Here
// the state, its spectrum and the field never leave LDS, a thread keeps its cell's m_n and
// accumulator and its frequency pairs' entries of the octant in registers from the first
// stage to the last, and what remains is the chain of a stage: x lines, y lines, product and
// back, some dozen barriers.  Measured per RK4 step with graph replay, two launches -> this:
// FP32 8x8x1 28.4 -> 15.5 us, 32x8x1 30.4 -> 24.7, 16x16x1 30.8 -> 26.4, 20x20x1 44.2 -> 26.8,
// 27x18x1 45.5 -> 30.2; FP64 8x8x1 34.2 -> 20.4.  With the radices of the separate passes (16 in
// one stage) 8x8x1 took 21.3 us and 20x20x1 30.9.
#include <algorithm>

#include "mm_llg_body.hpp"
#include "mm_rline.hpp"

namespace mm {

constexpr int kTinyMaxThreads = 512;
constexpr int kTinyRadix = 8;               // radices up to
constexpr int kTinyPairs = 2;               // frequency pairs a thread takes
constexpr size_t kTinyLds = 64 * 1024;
constexpr int64_t kTinyStepsPerLaunch = 4096;  // 63 to 124 ms at 15.5 to 30.2 us a step

// LDS: the stage input and the demag field [3][2 np][nx + 1] (np = ceil(ny / 2) row pairs; the
// last column and an odd grid's last row read as zero), the x lines [3][np], the spectrum
// [3][hx][Py], the stage twiddles of both lengths.
static size_t tiny_lds_bytes(int nx, int ny, int Px, int Py, size_t esz)
{
    const size_t np = (size_t)(ny + 1) / 2, cells = 3 * 2 * np * (size_t)(nx + 1);
    return (2 * (3 * np * rline_len(Px) + 3 * (size_t)(Px / 2 + 1) * rline_len(Py) + Px + Py) + 2 * cells) * esz;
}

// The twiddles of a schedule's stages, exp(-2 pi i r k / (span R)), from those of its length.
template <typename T>
__device__ inline void tiny_twiddles(const LinePlan& s, const cpx<T>* __restrict__ w, cpx<T>* out)
{
    for (int q = 1; q < s.ns; ++q) {
        const int span = s.p[q], n = (s.R[q] - 1) * span, step = s.P / (span * s.R[q]);
        for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) {
            const int r = i / span;
            out[s.toff[q] + i] = w[(r + 1) * (i - r * span) * step];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(kTinyMaxThreads) void k_tiny_steps(TinyArgs<T> g, LinePlan plx, LinePlan ply)
{
    extern __shared__ __attribute__((aligned(16))) char tiny_smem[];
    const LineRegs sx(plx), sy(ply);
    const LlgArgs<T>& a = g.g;
    const int Px = sx.P, Py = sy.P, LX = rline_len(Px), LY = rline_len(Py), hx = Px / 2 + 1, H1 = Py / 2 + 1;
    const int nx = a.nx, ny = a.ny, np = (ny + 1) / 2, W = nx + 1, CS = 2 * np * W, SC = hx * LY;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    cpx<T>* xl = reinterpret_cast<cpx<T>*>(tiny_smem);
    cpx<T>* S = xl + 3 * np * LX;
    cpx<T>*twx = S + 3 * SC, *twy = twx + Px;
    T* mc = reinterpret_cast<T*>(twy + Py);
    T* hd = mc + 3 * CS;
    tiny_twiddles<T>(plx, (const cpx<T>*)g.twx, twx);
    tiny_twiddles<T>(ply, (const cpx<T>*)g.twy, twy);

    // ---- this thread's cell, frequency pairs and x line
    const int64_t N = a.N;
    const bool own = t < (int)N;
    const int cj = own ? t / nx : 0, ci = own ? t - cj * nx : 0, at = cj * W + ci;
    const int dxm = ci > 0 ? -1 : 0, dxp = ci < nx - 1 ? 1 : 0, dym = cj > 0 ? -W : 0, dyp = cj < ny - 1 ? W : 0;
    const T kan = a.ku ? a.ku[own ? t : 0] : a.can;
    T mn[3], acc[3] = {(T)0, (T)0, (T)0};
#pragma unroll
    for (int d = 0; d < 3; ++d) mn[d] = g.m[d * N + (own ? t : 0)];
    T kv[kTinyPairs][4];
#pragma unroll
    for (int it = 0; it < kTinyPairs; ++it) {
        const int idx = min(t + it * NT, hx * H1 - 1);
#pragma unroll
        for (int c = 0; c < 4; ++c) kv[it][c] = ((const T*)g.kern)[c * g.k_cs + idx];
    }
    const LaneOf w = rline_lane(sx, 3 * np);
    const int xc = w.l / np, xp = w.l - xc * np;  // component, row pair
    cpx<T>* xln = xl + w.l * LX;
    T* mrow = mc + xc * CS + 2 * xp * W;
    T* hrow = hd + xc * CS + 2 * xp * W;
    const cpx<T>* srow = S + xc * SC + 2 * xp;
    const bool two = 2 * xp + 1 < ny;
    for (int i = t; i < 3 * CS; i += NT) mc[i] = (T)0;
    __syncthreads();
    if (own) {
#pragma unroll
        for (int d = 0; d < 3; ++d) mc[d * CS + at] = mn[d];
    }
    __syncthreads();

    const int yper = NT / sy.TL;
    for (int64_t step = 0; step < g.nsteps; ++step) {
        for (int stage = 1; stage <= 4; ++stage) {
            // ---- x forward of the row pairs, half spectra transposed into S
            rline_fft<T, kTinyRadix, false, true>(
                sx, twx, xln, w.u, w.real,
                [&](int e) {
                    const int i = e < nx ? e : nx;
                    return cpx<T>{mrow[i], mrow[W + i]};
                },
                [&](int e, cpx<T> v) { xln[e] = v; });
            __syncthreads();
            for (int idx = t; idx < 3 * np * hx; idx += NT) {
                const int q = div_by(idx, g.hmul), kx = idx - q * hx;
                const int c = np == 1 ? q : div_by(q, g.npmul), p = q - c * np;
                const cpx<T>* l = xl + q * LX;
                const cpx<T> zk = l[kx], zm = l[kx == 0 ? 0 : Px - kx];
                // Z = FFT(a + i b): A = (Z_k + conj Z_-k)/2, B = (Z_k - conj Z_-k)/(2i)
                cpx<T>* o = S + c * SC + kx * LY + 2 * p;
                o[0] = scale(zk + conj(zm), (T)0.5);
                if (2 * p + 1 < ny) o[1] = scale(mul_mi(zk - conj(zm)), (T)0.5);
            }
            __syncthreads();
            // ---- y forward, the Eq. 14 product, y inverse (conjugated)
            for (int q0 = 0; q0 < 3 * hx; q0 += yper) {
                const LaneOf v = rline_lane(sy, min(yper, 3 * hx - q0));
                cpx<T>* ln = S + (q0 + v.l) * LY;
                rline_fft<T, kTinyRadix, true, true>(
                    sy, twy, ln, v.u, v.real, [&](int e) { return e < ny ? ln[e] : cpx<T>{(T)0, (T)0}; },
                    [&](int e, cpx<T> x) { ln[e] = x; });
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < kTinyPairs; ++it) {
                const int idx = t + it * NT;
                if (idx < hx * H1) {
                    const int kx = div_by(idx, g.h1mul), ky = idx - kx * H1;
                    const bool mirror = ky > 0 && 2 * ky < Py;
                    cpx<T>* q = S + kx * LY;
                    thin_product(q + ky, q + (mirror ? Py - ky : ky), mirror, SC, kv[it][0], kv[it][1], kv[it][2],
                                 kv[it][3]);
                }
            }
            __syncthreads();
            for (int q0 = 0; q0 < 3 * hx; q0 += yper) {
                const LaneOf v = rline_lane(sy, min(yper, 3 * hx - q0));
                cpx<T>* ln = S + (q0 + v.l) * LY;
                rline_fft<T, kTinyRadix, true, true>(
                    sy, twy, ln, v.u, v.real, [&](int e) { return ln[e]; }, [&](int e, cpx<T> x) { ln[e] = x; });
            }
            __syncthreads();
            // ---- x inverse of the row pairs (S holds conjugates) into the field
            rline_fft<T, kTinyRadix, false, false>(
                sx, twx, xln, w.u, w.real,
                [&](int k) {
                    const bool lo = k < hx;
                    const cpx<T>* s = srow + (lo ? k : Px - k) * LY;
                    cpx<T> A = conj(s[0]), B = conj(s[two ? 1 : 0]);
                    if (!two) B = cpx<T>{(T)0, (T)0};
                    if (k == 0 || 2 * k == Px) A.im = B.im = (T)0;  // DC and Nyquist bins of a real row are real
                    return lo ? cpx<T>{A.re - B.im, -A.im - B.re} : cpx<T>{A.re + B.im, A.im - B.re};
                },
                [&](int e, cpx<T> v) {  // result a + i b = conj(v); what is cut off goes to column nx
                    const int i = e < nx ? e : nx;
                    hrow[i] = v.re;
                    hrow[W + i] = -v.im;
                });
            __syncthreads();
            // ---- the stage update of the thread's cell (llg_cell, in registers)
            T res[3];
            {
                T m[3], lap[3], h[3], F[3], heff[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const T* u = mc + d * CS + at;
                    const T c = u[0];
                    T s = (T)0;
                    s += u[dxm] - c;
                    s += u[dxp] - c;
                    s += u[dym] - c;
                    s += u[dyp] - c;
                    m[d] = c;
                    lap[d] = s;
                    h[d] = hd[d * CS + at];
                }
                llg_increment<T>(a, m, lap, h, kan, F, heff);
                if (stage == 1) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        acc[d] = F[d];
                        res[d] = m[d] + (T)0.5 * F[d];
                    }
                } else if (stage < 4) {
                    const T wt = stage == 2 ? (T)0.5 : (T)1;
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        acc[d] = acc[d] + (T)2 * F[d];
                        res[d] = mn[d] + wt * F[d];
                    }
                } else {
                    T v[3];
#pragma unroll
                    for (int d = 0; d < 3; ++d) v[d] = mn[d] + (acc[d] + F[d]) / (T)6;
                    const T inv = (T)1 / sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
#pragma unroll
                    for (int d = 0; d < 3; ++d) mn[d] = res[d] = v[d] * inv;
                }
            }
            __syncthreads();  // every neighbour is read
            if (own) {
#pragma unroll
                for (int d = 0; d < 3; ++d) mc[d * CS + at] = res[d];
            }
            __syncthreads();
        }
    }
    if (own) {
#pragma unroll
        for (int d = 0; d < 3; ++d) g.m[d * N + t] = mn[d];
    }
}

int tiny_plan(int nx, int ny, int Px, int Py, size_t esz, LinePlan* x, LinePlan* y)
{
    if (2 * nx > Px + 1 || 2 * ny > Py + 1) return 0;
    const int np = (ny + 1) / 2, hx = Px / 2 + 1, pairs = hx * (Py / 2 + 1);
    // One CU works where the passes have many, so the line lies at the entries of a spectrum,
    // hx Py: FP32 27x18x1 (1008) 45.5 -> 30.2 us, but 22x23x1 (1035) 45.4 -> 45.5, 32x16x1
    // (1056) 31.7 -> 40.0, 8x60x1 (1080) 38.4 -> 42.3; FP64 8x8x1 (144) 34.2 -> 20.4, but
    // 32x8x1 (528) 36.6 -> 36.2, 16x16x1 (544) 35.3 -> 38.9.
    if (hx * Py > (esz == 8 ? 256 : 1024)) return 0;
    if (!make_line_plan(Px, x, 3 * np, kTinyMaxThreads) || !make_line_plan(Py, y, 3 * hx, kTinyMaxThreads)) return 0;
    if (y->TL > kTinyMaxThreads) return 0;
    const int lines = std::max(3 * np * x->TL, std::min(kTinyMaxThreads / y->TL, 3 * hx) * y->TL);
    const int nt = (std::max(std::max(nx * ny, lines), (pairs + kTinyPairs - 1) / kTinyPairs) + 63) / 64 * 64;
    return nt <= kTinyMaxThreads && tiny_lds_bytes(nx, ny, Px, Py, esz) <= kTinyLds ? nt : 0;
}

template <typename T>
hipError_t launch_tiny_steps(TinyArgs<T> a, int64_t nsteps, const LinePlan& x, const LinePlan& y, int nt,
                             hipStream_t st)
{
    const int nx = a.g.nx, ny = a.g.ny;
    const size_t lds = tiny_lds_bytes(nx, ny, x.P, y.P, sizeof(T));
    if (nt < 1 || nt > kTinyMaxThreads || lds > kTinyLds || a.g.nz != 1 || a.g.per != 0 || a.ncomp != 4)
        return hipErrorInvalidValue;
    a.hmul = div_mul(x.P / 2 + 1);
    a.h1mul = div_mul(y.P / 2 + 1);
    a.npmul = div_mul((ny + 1) / 2);
    for (int64_t n = 0; n < nsteps; n += a.nsteps) {
        a.nsteps = std::min(nsteps - n, kTinyStepsPerLaunch);
        hipLaunchKernelGGL(k_tiny_steps<T>, dim3(1), dim3(nt), lds, st, a, x, y);
    }
    return hipGetLastError();
}
#define MM_INST(T) \
    template hipError_t launch_tiny_steps<T>(TinyArgs<T>, int64_t, const LinePlan&, const LinePlan&, int, hipStream_t);
MM_INST(float)
MM_INST(double)
#undef MM_INST

}  // namespace mm
