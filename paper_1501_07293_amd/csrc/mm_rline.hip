// mm_rline.hip -- kernels of the runtime-length register passes (bodies in
// mm_rline.hpp), the choice of a line's radices and of the work-group shapes.
#include <algorithm>

#include "mm_rline.hpp"

namespace mm {

constexpr int kRMaxThreads = 512;

extern __shared__ __align__(16) char rline_smem[];

template <typename T, int RM>
__global__ __launch_bounds__(kRMaxThreads) void k_rxfwd(RXArgs a, LinePlan s)
{
    body_rxfwd<T, RM>(a, s, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}
template <typename T, int RM>
__global__ __launch_bounds__(kRMaxThreads) void k_rxinv(RXArgs a, LinePlan s)
{
    body_rxinv<T, RM>(a, s, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}
template <typename T, int RM, bool INV>
__global__ __launch_bounds__(kRMaxThreads) void k_ryline(RYArgs a, LinePlan s)
{
    body_ryline<T, RM, INV>(a, s, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}
template <typename T, int RM>
__global__ __launch_bounds__(kRMaxThreads) void k_rkz(RKzArgs a, LinePlan s)
{
    body_rkz<T, RM>(a, s, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}
template <typename T, int RM>
__global__ __launch_bounds__(kRMaxThreads) void k_rky(RKyArgs a, LinePlan s)
{
    body_rky<T, RM>(a, s, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}

// FP32 work-groups of up to 1024 threads (128 registers a thread hold every radix)
template <typename T>
constexpr int ryz_max_threads() { return sizeof(T) == 4 ? 1024 : kRMaxThreads; }

template <typename T, int RM>
__global__ __launch_bounds__(ryz_max_threads<T>()) void k_ryz(RYzArgs a, LinePlan y, LinePlan z)
{
    body_ryz<T, RM>(a, y, z, xcd_tile(blockIdx.x, gridDim.x), reinterpret_cast<cpx<T>*>(rline_smem));
}

// p[i] = exp(-2 pi i r k / (span R)) for the entry's stage, r and k
template <typename T>
__global__ void k_stage_twiddles(cpx<T>* out, LinePlan s)
{
    const int n = s.P - s.R[0];
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        int q = 1;
        while (q + 1 < s.ns && i >= s.toff[q + 1]) ++q;
        const int j = i - s.toff[q], r = j / s.p[q] + 1, k = j % s.p[q];
        double sn, cs;
        sincospi(-2.0 * (double)((long long)r * k) / (double)(s.p[q] * s.R[q]), &sn, &cs);
        out[i] = cpx<T>{(T)cs, (T)sn};
    }
}

template <typename T>
hipError_t launch_stage_twiddles(void* tws, const LinePlan& s, hipStream_t st)
{
    const int n = s.ns > 0 ? s.P - s.R[0] : 0;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_stage_twiddles<T>, dim3((n + 255) / 256), dim3(256), 0, st, (cpx<T>*)tws, s);
    return hipGetLastError();
}

// ------------------------------------------------------------------ schedules
// Instructions of one radix butterfly, roughly (its DFT, its twiddles, its LDS and
// address work), and of a stage's barriers per thread.
static double radix_cost(int R, bool first)
{
    static const double dft[17] = {0, 0, 4, 14, 16, 40, 40, 72, 56, 76, 100, 104, 0, 0, 172, 170, 176};
    double d = R == 12 ? 104 : dft[R];
    d += first ? 6.0 * R : 6.0 * R + 6.0 * (R - 1);
    // the first stage's LDS stores run with stride R: two-way bank conflicts from a
    // factor 4, four-way from 8, eight-way from 16
    if (first) d += R % 16 == 0 ? 14.0 * R : (R % 8 == 0 ? 6.0 * R : (R % 4 == 0 ? 2.0 * R : 0.0));
    return d;
}

// lines > 0: for that many lines side by side in one work-group of up to max_threads, with
// radices up to 8: what counts is a thread's chain, times the rounds the lines take.
bool make_line_plan(int P, LinePlan* s, int lines, int max_threads)
{
    *s = LinePlan{};
    if (P < 2 || P > 8192) return false;
    static const int set[] = {16, 15, 14, 12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
    int cur[kMaxLineStages], best[kMaxLineStages], nbest = 0;
    double cbest = 1e300;
    // every ordered factorisation into radices of the set; a thread of the line runs
    // every stage, so a stage costs its butterfly whatever share of the threads works
    auto rec = [&](auto&& self, int rest, int n) -> void {
        if (rest == 1) {
            int rmin = cur[0];
            for (int i = 1; i < n; ++i) rmin = cur[i] < rmin ? cur[i] : rmin;
            double c = 0;
            for (int i = 0; i < n; ++i) c += radix_cost(cur[i], i == 0 && n > 1) + 40.0;
            if (lines > 0)
                c *= (lines * (P / rmin) + max_threads - 1) / max_threads;
            else
                c *= (double)(P / rmin) / P;
            if (c < cbest) {
                cbest = c;
                nbest = n;
                for (int i = 0; i < n; ++i) best[i] = cur[i];
            }
            return;
        }
        if (n == kMaxLineStages) return;
        for (int r : set)
            if (rest % r == 0 && (lines <= 0 || r <= 8)) {
                cur[n] = r;
                self(self, rest / r, n + 1);
            }
    };
    rec(rec, P, 0);
    if (nbest == 0) return false;
    s->P = P;
    s->ns = nbest;
    int span = 1, off = 0;
    for (int q = 0; q < nbest; ++q) {
        s->R[q] = best[q];
        s->p[q] = span;
        s->m[q] = P / best[q];
        s->pmul[q] = div_mul(span);
        s->toff[q] = off;
        if (q > 0) off += (best[q] - 1) * span;
        if (s->m[q] > s->TL) s->TL = s->m[q];
        span *= best[q];
    }
    s->tmul = div_mul(s->TL);
    return true;
}

constexpr size_t kRLdsBudget = 64 * 1024;  // dynamic LDS of a work-group

size_t rline_lds_bytes(int lines, int P, size_t esz) { return (size_t)lines * rline_len(P) * 2 * esz; }
size_t ryz_lds_bytes(int Py, int Pz, size_t esz) { return (size_t)3 * Pz * rline_len(Py) * 2 * esz; }
size_t rxinv_lds_bytes(int lsh, int P, size_t esz)
{
    const size_t lines = rline_lds_bytes(1 << lsh, P, esz), raw = (size_t)(2 << lsh) * (P / 2 + 1) * 2 * esz;
    return lines > raw ? lines : raw;
}

RShape rline_shapes(const LinePlan& x, const LinePlan& y, const LinePlan& z, int nx, int ny, int nz, size_t esz,
                    int max_threads, int min_groups)
{
    RShape r{-1, -1, 0, 0, 0, -1, 0};
    const int pairs = (ny + 1) / 2;
    if (x.ns > 0) {
        // 128-byte transposed segments (8 row pairs in FP32, 4 in FP64), more where a
        // line takes few threads, fewer while the launch has under 256 work-groups
        auto lines = [&](bool inverse) {
            auto fits = [&](int l) {
                return (x.TL << l) <= max_threads &&
                       (inverse ? rxinv_lds_bytes(l, x.P, esz) : rline_lds_bytes(1 << l, x.P, esz)) <= kRLdsBudget;
            };
            int l = esz == 8 ? 2 : 3;
            while (l < 4 && (x.TL << l) < 128) ++l;
            while (l > 0 && (!fits(l) || 3 * nz * ((pairs + (1 << l) - 1) >> l) < min_groups)) --l;
            return fits(l) ? l : -1;
        };
        r.lsh_f = lines(false);
        r.lsh_i = lines(true);
    }
    if (y.ns > 0) {
        const int cap = (int)(kRLdsBudget / rline_lds_bytes(1, y.P, esz));
        int l = 256 / y.TL;
        if (l < 1 && y.TL <= max_threads) l = 1;
        r.y = l < cap ? l : cap;
        const int hx = x.P / 2 + 1;
        l = 256 / (3 * y.TL);
        if (l < 1 && 3 * y.TL <= max_threads) l = 1;
        while (l > 1 && (hx + l - 1) / l < min_groups) --l;
        r.ky = 3 * l <= cap ? l : cap / 3;
        l = 256 / (6 * y.TL);
        if (l < 1 && 6 * y.TL <= max_threads) l = 1;
        while (l > 1 && (hx + l - 1) / l < min_groups) --l;
        r.ky2 = 6 * l <= cap ? l : cap / 6;
        if (6 * (int64_t)hx * ny * 2 * (int64_t)esz >= kBufEnd) r.ky = r.ky2 = 0;
    }
    if (z.ns > 0) {
        const int64_t ncols = (int64_t)(x.P / 2 + 1) * y.P;
        int c = 6;
        auto fits = [&](int q) {
            return (3 * z.TL << q) <= max_threads && rline_lds_bytes(3 << q, z.P, esz) <= kRLdsBudget;
        };
        while (c > 0 && (!fits(c) || ((3 * z.TL << c) > 256 && c > 4))) --c;
        // the pass addresses the whole spectrum from one descriptor, and the octant from another
        const int64_t oct = 6 * (int64_t)(z.P / 2 + 1) * (x.P / 2 + 1) * (y.P / 2 + 1) * (int64_t)esz;
        if (fits(c) && 3 * nz * ncols * 2 * (int64_t)esz < kBufEnd && oct < kBufEnd) r.csh = c;
    }
    if (y.ns > 0 && z.ns > 0 && nz > 1 && y.TL <= kRMaxThreads && z.TL <= kRMaxThreads &&
        ryz_lds_bytes(y.P, z.P, esz) <= kLdsBudget &&
        3 * (int64_t)nz * (x.P / 2 + 1) * y.P * 2 * (int64_t)esz < kRLineBytes) {
        // as many threads as the longer of the two line sets takes: there are about as
        // many bins as CUs or fewer, so what counts is the number of rounds
        const int cap = esz == 4 ? 1024 : kRMaxThreads;
        const int want = std::max(3 * nz * y.TL, 3 * y.P * z.TL);
        r.yz = std::min(cap, std::max(256, (want + 63) / 64 * 64));
    }
    return r;
}

// the instantiation that serves every radix of s
static bool small_radices(const LinePlan& s)
{
    for (int q = 0; q < s.ns; ++q)
        if (s.R[q] > 10) return false;
    return true;
}
#define MM_RLAUNCH(k10, k16, grid, nt, lds, st, ...)                                            \
    do {                                                                                        \
        if (small_radices(s))                                                                   \
            hipLaunchKernelGGL(k10, dim3(grid), dim3(nt), lds, st, __VA_ARGS__);                \
        else                                                                                    \
            hipLaunchKernelGGL(k16, dim3(grid), dim3(nt), lds, st, __VA_ARGS__);                \
    } while (0)

static int round64(int n) { return (n + 63) / 64 * 64; }

template <typename T>
hipError_t launch_rxline(const RXArgs& a, const LinePlan& s, int inverse, hipStream_t st)
{
    const int rows = 2 << a.lsh, grid = a.nplanes * ((a.ny + rows - 1) / rows), nt = round64(s.TL << a.lsh);
    if (nt > kRMaxThreads) return hipErrorInvalidValue;
    if (grid <= 0) return hipSuccess;
    if (inverse)
        MM_RLAUNCH((k_rxinv<T, 10>), (k_rxinv<T, 16>), grid, nt, rxinv_lds_bytes(a.lsh, s.P, sizeof(T)), st, a, s);
    else
        MM_RLAUNCH((k_rxfwd<T, 10>), (k_rxfwd<T, 16>), grid, nt, rline_lds_bytes(1 << a.lsh, s.P, sizeof(T)), st, a, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ryline(const RYArgs& a, const LinePlan& s, int inverse, hipStream_t st)
{
    const int grid = (a.nlines + a.L - 1) / a.L, nt = round64(s.TL * a.L);
    const size_t lds = rline_lds_bytes(a.L, s.P, sizeof(T));
    if (nt > kRMaxThreads) return hipErrorInvalidValue;
    if (grid <= 0) return hipSuccess;
    if (inverse)
        MM_RLAUNCH((k_ryline<T, 10, true>), (k_ryline<T, 16, true>), grid, nt, lds, st, a, s);
    else
        MM_RLAUNCH((k_ryline<T, 10, false>), (k_ryline<T, 16, false>), grid, nt, lds, st, a, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rkz(const RKzArgs& a, const LinePlan& s, hipStream_t st)
{
    const int C = 1 << a.csh, grid = (a.ncols + C - 1) / C, nt = round64(3 * s.TL * C);
    if (nt > kRMaxThreads) return hipErrorInvalidValue;
    if (grid <= 0) return hipSuccess;
    MM_RLAUNCH((k_rkz<T, 10>), (k_rkz<T, 16>), grid, nt, rline_lds_bytes(3 * C, s.P, sizeof(T)), st, a, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_rky(const RKyArgs& a, const LinePlan& s, hipStream_t st)
{
    const int grid = (a.hx + a.L - 1) / a.L, nt = round64(3 * s.TL * a.L);
    if (nt > kRMaxThreads) return hipErrorInvalidValue;
    if (grid <= 0) return hipSuccess;
    MM_RLAUNCH((k_rky<T, 10>), (k_rky<T, 16>), grid, nt, rline_lds_bytes(3 * a.L, s.P, sizeof(T)), st, a, s);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ryz(const RYzArgs& a, const LinePlan& y, const LinePlan& z, hipStream_t st)
{
    const size_t lds = ryz_lds_bytes(y.P, z.P, sizeof(T));
    if (a.nt > ryz_max_threads<T>() || y.TL > a.nt || a.zper < 1 || a.zper * z.TL > a.nt || lds > (size_t)kLdsBudget)
        return hipErrorInvalidValue;
    if (a.hx <= 0) return hipSuccess;
    auto go = [&](auto kern) {
        if (lds > kRLdsBudget) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kern, dim3(a.hx), dim3(a.nt), lds, st, a, y, z);
        return hipGetLastError();
    };
    return small_radices(y) && small_radices(z) ? go(k_ryz<T, 10>) : go(k_ryz<T, 16>);
}

#define MM_INST(T)                                                                       \
    template hipError_t launch_stage_twiddles<T>(void*, const LinePlan&, hipStream_t);   \
    template hipError_t launch_rxline<T>(const RXArgs&, const LinePlan&, int, hipStream_t); \
    template hipError_t launch_ryline<T>(const RYArgs&, const LinePlan&, int, hipStream_t); \
    template hipError_t launch_rkz<T>(const RKzArgs&, const LinePlan&, hipStream_t);     \
    template hipError_t launch_rky<T>(const RKyArgs&, const LinePlan&, hipStream_t);     \
    template hipError_t launch_ryz<T>(const RYzArgs&, const LinePlan&, const LinePlan&, hipStream_t);
MM_INST(float)
MM_INST(double)
#undef MM_INST

}  // namespace mm
