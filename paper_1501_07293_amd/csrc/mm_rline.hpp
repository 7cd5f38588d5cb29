// mm_rline.hpp -- FFT passes of any 7-smooth padded length, with the length a
// runtime value and the transforms in registers.
//
// A line of P points is worked by TL = P / (its smallest radix) threads, one
// butterfly per thread and stage: the radices of a LinePlan (2 .. 16, composites
// such as 6, 10, 12, 14 and 15 included, so lengths up to 256 take one or two stages, a dozen
// of them three to five, and up to 4096 mostly three) are chosen on the host, and each stage switches on its radix
// (the same for the whole work-group) to a body unrolled for it.  The first stage
// takes its inputs straight from where they are (global memory, or LDS for an inverse
// after the k-space product), the stages between exchange through LDS, and the last
// one hands its outputs to the caller.  Every index is linear in the stage's loop
// variable (one addition an element, no division inside a stage), and the twiddles of
// a stage lie [r][k] so that consecutive threads read consecutive entries.
//
// What these replace ran every length through one LDS-staged body with 16 elements a
// thread: a division and a remainder per element to find its line, 215 to 233
// registers (two waves a SIMD) and strided twiddle reads.  Measured per RK4 step, all passes
// of a stage together (and with the fused stage and plane passes where they apply), before ->
// now: 200x200x1 FP32 237 -> 80 us, FP64 261 -> 93; 100x100x10 368 -> 121 and 495 -> 169;
// 301x190x6 729 -> 228 and 1155 -> 327; 360x300x10 periodic in x and y 655 -> 269 and 1031 ->
// 435; 96x96x96 880 -> 490 and 1687 -> 861.  What bounds them now: on grids of some 10^5 cells
// the latency of their dependent launches and LDS stages, on the larger ones the caches and
// memory (the stage update beside them runs at the copy rate there).
//
// Spectrum layout: as everywhere, S = [3][nz][hx][Sy].
#pragma once
#include "mm_fast.hpp"
#include "mm_kernels.hpp"

namespace mm {

// ------------------------------------------------------------------ the line
// LDS length of a line: odd, so that consecutive lines start on different banks.
__host__ __device__ constexpr int rline_len(int P) { return P | 1; }

// n / d for 0 <= n < 2^16 and 1 < d < 2^16, by the multiplier floor(2^32 / d) + 1
__device__ inline int div_by(int n, unsigned mul) { return (int)__umulhi((unsigned)n, mul); }

// A schedule in scalar registers: every field is read once, at a constant index (a
// dynamic one would copy the schedule to private memory), before the first barrier, so
// that the switch on a stage's radix is a scalar branch and no stage waits for its
// schedule.
__device__ inline int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }
struct LineStage {
    int R, p, m, toff;
    unsigned pmul;
};
struct LineRegs {
    int P, ns, TL;
    unsigned tmul;
    LineStage s0, s1, s2, s3, s4;  // named, not an array: every access is a register
    static __device__ inline LineStage load(const LinePlan& s, int q)
    {
        return LineStage{sgpr(s.R[q]), sgpr(s.p[q]), sgpr(s.m[q]), sgpr(s.toff[q]), (unsigned)sgpr((int)s.pmul[q])};
    }
    __device__ inline explicit LineRegs(const LinePlan& s)
        : P(sgpr(s.P)), ns(sgpr(s.ns)), TL(sgpr(s.TL)), tmul((unsigned)sgpr((int)s.tmul)), s0(load(s, 0)),
          s1(load(s, 1)), s2(load(s, 2)), s3(load(s, 3)), s4(load(s, 4))
    {
        static_assert(kMaxLineStages == 5, "stages named by hand");
    }
    __device__ inline LineStage stage(int q) const
    {
        // by value through readfirstlane: a choice between the fields' addresses would
        // put the schedule into private memory
        auto pick = [q](int a0, int a1, int a2, int a3, int a4) {
            a0 = sgpr(a0), a1 = sgpr(a1), a2 = sgpr(a2), a3 = sgpr(a3), a4 = sgpr(a4);
            return q == 0 ? a0 : (q == 1 ? a1 : (q == 2 ? a2 : (q == 3 ? a3 : a4)));
        };
        return LineStage{pick(s0.R, s1.R, s2.R, s3.R, s4.R), pick(s0.p, s1.p, s2.p, s3.p, s4.p),
                         pick(s0.m, s1.m, s2.m, s3.m, s4.m), pick(s0.toff, s1.toff, s2.toff, s3.toff, s4.toff),
                         (unsigned)pick((int)s0.pmul, (int)s1.pmul, (int)s2.pmul, (int)s3.pmul, (int)s4.pmul)};
    }
};

// The radices a kernel serves: all, or (RM = 10) those up to 10, whose butterflies need
// about 40 registers fewer.
#define MM_RADIX_CASES(X)                                         \
    X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)                 \
    X(12) X(14) X(15) X(16)

// An entry of a stage table: row (the same for every thread) plus a byte offset below
// 4 GiB, so that the load takes its base from scalar registers.
template <typename T>
__device__ inline cpx<T> ld_tw(const cpx<T>* row, unsigned bytes)
{
    return *reinterpret_cast<const cpx<T>*>(reinterpret_cast<const char*>(row) + bytes);
}

// This thread's line (of `lines` side by side) and its number u in it.  A thread past the
// last line takes the part of thread 0 of line 0 (real = false), so that it reads and
// writes valid LDS: what it writes there is what that thread writes.
struct LaneOf {
    int l, u;
    bool real;
};
__device__ inline LaneOf rline_lane(const LineRegs& s, int lines)
{
    const int t = (int)threadIdx.x;
    const int l = s.TL == 1 ? t : div_by(t, s.tmul);
    const bool real = l < lines;
    return LaneOf{real ? l : 0, real ? t - l * s.TL : 0, real};
}

// Forward FFT of one line by its TL threads; u and real as LaneOf.  get(e) delivers input
// e of the first stage; put(e, value) takes output e.  Both are called by every thread and
// must not branch.  PUT_LDS: put writes to the line's own LDS entry e; otherwise to global
// memory, and threads without a butterfly pass an e of kPastEnd or more, which has to
// store nothing.  SYNC: the inputs come from LDS that the stages overwrite, so every
// thread's reads end before the first write.  tws: the line's stage twiddles.
//
// A stage with fewer butterflies than the line has threads gives the others butterfly 0
// again.  So a radix case is straight-line code that ends in its own stores: with a
// divergent branch in it, or with its values handed to code behind the switch, the
// compiler keeps the values of all cases side by side (up to 256 registers, spilled).
constexpr int kPastEnd = 0x40000000;

// ES: entries from one element of the line to the next in LDS (0: es, a run-time value).
template <typename T, int RM, bool SYNC, bool PUT_LDS, int ES = 1, class Get, class Put>
__device__ __forceinline__ void rline_fft(const LineRegs& s, const cpx<T>* __restrict__ tws, cpx<T>* ln, int u, bool real,
                                          Get get, Put put, int es = 1)
{
    const int ns = s.ns;
    if constexpr (ES != 0) es = ES;
    {
        const int m = s.s0.m;
        const int i = u < m ? u : 0;
        const int io = PUT_LDS || (real && u < m) ? i : kPastEnd;
        switch (s.s0.R) {
#define X(RR)                                                                         \
    case RR:                                                                          \
        if constexpr (RR <= RM) {                                                     \
            cpx<T> v[RR];                                                             \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) v[r] = get(i + r * m);     \
            Dft<T, RR>::run(v);                                                       \
            if (SYNC) __syncthreads();                                                \
            if (ns == 1) {                                                            \
                _Pragma("unroll") for (int r = 0; r < RR; ++r) put(io + r, v[r]);     \
            } else {                                                                  \
                cpx<T>* o = ln + i * RR * es;                                         \
                _Pragma("unroll") for (int r = 0; r < RR; ++r) o[r * es] = v[r];      \
            }                                                                         \
        }                                                                             \
        break;
            MM_RADIX_CASES(X)
#undef X
        default: break;
        }
        if (ns == 1) return;
        __syncthreads();
    }
    for (int q = 1; q < ns - 1; ++q) {
        const LineStage c = s.stage(q);
        const int m = c.m, p = c.p;
        const int i = u < m ? u : 0;
        const int k = i - div_by(i, c.pmul) * p;
        const cpx<T>* w = tws + c.toff;
        const unsigned kb = (unsigned)k * (unsigned)sizeof(cpx<T>);
        switch (c.R) {
#define X(RR)                                                                                 \
    case RR:                                                                                  \
        if constexpr (RR <= RM) {                                                             \
            cpx<T> v[RR], tw[RR];                                                             \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) tw[r] = ld_tw(w + (r - 1) * p, kb); \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) v[r] = ln[(i + r * m) * es];       \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) v[r] = cmul(v[r], tw[r]);          \
            Dft<T, RR>::run(v);                                                               \
            __syncthreads();                                                                  \
            cpx<T>* o = ln + ((i - k) * RR + k) * es;                                         \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) o[r * p * es] = v[r];              \
        }                                                                                     \
        break;
            MM_RADIX_CASES(X)
#undef X
        default: break;
        }
        __syncthreads();
    }
    {
        // last stage: p = m, so k is i and the outputs sit where the inputs were
        const LineStage c = s.stage(ns - 1);
        const int m = c.m;
        const int i = u < m ? u : 0;
        const int io = PUT_LDS || (real && u < m) ? i : kPastEnd;
        const cpx<T>* w = tws + c.toff;
        const unsigned kb = (unsigned)i * (unsigned)sizeof(cpx<T>);
        // in place in LDS, a thread that repeats butterfly 0 must have read it before
        // the one that owns it writes
        switch (c.R) {
#define X(RR)                                                                                 \
    case RR:                                                                                  \
        if constexpr (RR <= RM) {                                                             \
            cpx<T> v[RR], tw[RR];                                                             \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) tw[r] = ld_tw(w + (r - 1) * m, kb); \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) v[r] = ln[(i + r * m) * es];       \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) v[r] = cmul(v[r], tw[r]);          \
            Dft<T, RR>::run(v);                                                               \
            if (PUT_LDS) __syncthreads();                                                     \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) put(io + r * m, v[r]);             \
        }                                                                                     \
        break;
            MM_RADIX_CASES(X)
#undef X
        default: break;
        }
    }
}

// ------------------------------------------------------------------ y lines
template <typename T, int RM, bool INV>
__device__ inline void body_ryline(const RYArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const LaneOf w = rline_lane(s, a.L);
    const int line = tile * a.L + w.l;
    const bool ok = line < a.nlines;
    // the line's place: in memory order the work-group's lines follow one another, bin by
    // bin (kx_major) they lie anywhere in the buffer
    constexpr unsigned CS = sizeof(cpx<T>);
    const Buf g = buf_of((const cpx<T>*)a.buf + (a.kx_major ? 0 : (int64_t)tile * a.L * a.line_stride));
    int rel = w.l;
    if (a.kx_major) rel = (line % a.kx_major) * (a.nlines / a.kx_major) + line / a.kx_major;
    const unsigned at = (unsigned)rel * (unsigned)a.line_stride * CS;
    const int nin = ok ? a.nin : 0, nout = ok ? a.nout : 0;
    rline_fft<T, RM, false, false>(
        s, (const cpx<T>*)a.tws, lds + w.l * rline_len(s.P), w.u, w.real,
        [&](int e) {
            const cpx<T> x = buf_ld<cpx<T>>(g, e < nin ? at + (unsigned)e * CS : kBufNone);
            return INV ? conj(x) : x;
        },
        [&](int e, cpx<T> v) { buf_st(g, e < nout ? at + (unsigned)e * CS : kBufNone, INV ? conj(v) : v); });
}

// ------------------------------------------------------------------ x forward
// L = 1 << a.lsh complex lines (2 L consecutive rows of one plane) a work-group; the
// half spectrum is stored transposed, 2 L rows a bin.
template <typename T, int RM>
__device__ inline void body_rxfwd(const RXArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), hx = P / 2 + 1;
    const int L = 1 << a.lsh, rows = 2 * L;
    const int tpp = (a.ny + rows - 1) / rows;
    const int plane = tile / tpp, yb = (tile - plane * tpp) * rows;
    const LaneOf w = rline_lane(s, L);
    const int y0 = yb + 2 * w.l;
    const bool ok0 = y0 < a.ny, ok1 = y0 + 1 < a.ny;
    cpx<T>* ln = lds + w.l * LP;
    const int nx = a.nx;
    const Buf g = buf_of((const T*)a.in + ((int64_t)plane * a.ny + yb) * nx);
    const unsigned at0 = (unsigned)(2 * w.l * nx) * (unsigned)sizeof(T);
    const int n0 = ok0 ? nx : 0, n1 = ok1 ? nx : 0;
    rline_fft<T, RM, false, true>(
        s, (const cpx<T>*)a.tws, ln, w.u, w.real,
        [&](int e) {
            const T re = buf_ld<T>(g, e < n0 ? at0 + (unsigned)e * (unsigned)sizeof(T) : kBufNone);
            const T im = buf_ld<T>(g, e < n1 ? at0 + (unsigned)(nx + e) * (unsigned)sizeof(T) : kBufNone);
            return cpx<T>{re, im};
        },
        [&](int e, cpx<T> v) { ln[e] = v; });
    __syncthreads();
    cpx<T>* out = (cpx<T>*)a.out + (int64_t)plane * hx * a.srows;
    const bool paired = (a.srows & 1) == 0 && (reinterpret_cast<uintptr_t>(a.out) % sizeof(cpx2<T>)) == 0;
    for (int idx = threadIdx.x; idx < (hx << a.lsh); idx += blockDim.x) {
        const int q = idx & (L - 1), kx = idx >> a.lsh;
        const cpx<T> zk = lds[q * LP + kx];
        const cpx<T> zm = lds[q * LP + (kx == 0 ? 0 : P - kx)];
        // Z = FFT(a + i b): A = (Z_k + conj Z_-k)/2, B = (Z_k - conj Z_-k)/(2i)
        const cpx<T> A = scale(zk + conj(zm), (T)0.5);
        const cpx<T> B = scale(mul_mi(zk - conj(zm)), (T)0.5);
        const int y = yb + 2 * q;
        cpx<T>* o = out + (int64_t)kx * a.srows + y;
        if (paired && y + 1 < a.ny) {
            *reinterpret_cast<cpx2<T>*>(o) = cpx2<T>{A, B};
        } else {
            if (y < a.ny) o[0] = A;
            if (y + 1 < a.ny) o[1] = B;
        }
    }
}

// ------------------------------------------------------------------ x inverse
// The gather of the 2 L half-spectrum rows takes at most kRxGather bin pairs a thread
// (hx L of them over at least L P / R threads, R <= 16), all loaded before the first
// LDS store.
constexpr int kRxGather = 9;

template <typename T, int RM>
__device__ inline void body_rxinv(const RXArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), hx = P / 2 + 1;
    const int L = 1 << a.lsh, rows = 2 * L;
    const int tpp = (a.ny + rows - 1) / rows;
    const int plane = tile / tpp, yb = (tile - plane * tpp) * rows;
    const LaneOf w = rline_lane(s, L);
    const cpx<T>* src = (const cpx<T>*)a.in + (int64_t)plane * hx * a.srows;
    const int NT = blockDim.x, nel = hx << a.lsh;
    const bool paired = (a.srows & 1) == 0 && (reinterpret_cast<uintptr_t>(a.in) % sizeof(cpx2<T>)) == 0;
    cpx2<T> g[kRxGather];
#pragma unroll
    for (int it = 0; it < kRxGather; ++it) {
        const int idx = (int)threadIdx.x + it * NT;
        const int q = idx & (L - 1), kx = idx >> a.lsh, y = yb + 2 * q;
        g[it].a = g[it].b = cpx<T>{(T)0, (T)0};
        if (idx < nel) {
            const cpx<T>* p = src + (int64_t)kx * a.srows + y;
            if (paired && y + 1 < a.ny) {
                g[it] = *reinterpret_cast<const cpx2<T>*>(p);
            } else {
                if (y < a.ny) g[it].a = p[0];
                if (y + 1 < a.ny) g[it].b = p[1];
            }
        }
    }
#pragma unroll
    for (int it = 0; it < kRxGather; ++it) {
        const int idx = (int)threadIdx.x + it * NT;
        if (idx < nel) {
            const int q = idx & (L - 1), kx = idx >> a.lsh;
            lds[(2 * q) * hx + kx] = g[it].a;
            lds[(2 * q + 1) * hx + kx] = g[it].b;
        }
    }
    __syncthreads();
    const cpx<T>* ra = lds + 2 * w.l * hx;
    const cpx<T>* rb = ra + hx;
    const int y0 = yb + 2 * w.l, nx = a.nx;
    const int n0 = y0 < a.ny ? nx : 0, n1 = y0 + 1 < a.ny ? nx : 0;
    const Buf o = buf_of((const T*)a.out + ((int64_t)plane * a.ny + yb) * nx);
    const unsigned at0 = (unsigned)(2 * w.l * nx) * (unsigned)sizeof(T);
    rline_fft<T, RM, true, false>(
        s, (const cpx<T>*)a.tws, lds + w.l * LP, w.u, w.real,
        [&](int k) {
            const bool lo = k < hx;
            cpx<T> A = ra[lo ? k : P - k], B = rb[lo ? k : P - k];
            if (k == 0 || 2 * k == P) A.im = B.im = (T)0;  // DC and Nyquist bins of a real row are real
            // conj(A + i B) below hx, conj(conj A + i conj B) above: inverse by conjugation
            return lo ? cpx<T>{A.re - B.im, -A.im - B.re} : cpx<T>{A.re + B.im, A.im - B.re};
        },
        [&](int e, cpx<T> v) {  // result a + i b = conj(v)
            buf_st(o, e < n0 ? at0 + (unsigned)e * (unsigned)sizeof(T) : kBufNone, v.re);
            buf_st(o, e < n1 ? at0 + (unsigned)(nx + e) * (unsigned)sizeof(T) : kBufNone, -v.im);
        });
}

// ------------------------------------------------------------------ k-space
// Eq. 14 for one frequency: the three components at x, y, z in LDS times the real
// symmetric spectrum k (xx, xy, xz, yy, yz, zz), stored conjugated so that the inverse
// runs as a forward transform.
template <typename T>
__device__ inline void tensor_product(cpx<T>* px, cpx<T>* py, cpx<T>* pz, const T (&k)[6])
{
    const cpx<T> mx = *px, my = *py, mz = *pz;
    *px = conj(cpx<T>{k[0] * mx.re + k[1] * my.re + k[2] * mz.re, k[0] * mx.im + k[1] * my.im + k[2] * mz.im});
    *py = conj(cpx<T>{k[1] * mx.re + k[3] * my.re + k[4] * mz.re, k[1] * mx.im + k[3] * my.im + k[4] * mz.im});
    *pz = conj(cpx<T>{k[2] * mx.re + k[4] * my.re + k[5] * mz.re, k[2] * mx.im + k[4] * my.im + k[5] * mz.im});
}

// Frequency pairs k, P - k a thread takes (they share one octant entry up to the parities):
// C (P / 2 + 1) of them over at least 3 C P / R threads, R <= 16 and R <= P.
constexpr int kRzProduct = 3;

// Along z (3-D grids): C = 1 << a.csh adjacent columns (kx, ky), three component lines
// each; lanes run column-fastest, so a load or store of one z point is one segment of C
// columns and the octant loads of the product run along ky.
template <typename T, int RM>
__device__ inline void body_rkz(const RKzArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), C = 1 << a.csh;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const int l = t & (C - 1), v = t >> a.csh;  // v = component * TL + u
    int comp = s.TL == 1 ? v : div_by(v, s.tmul), u = v - comp * s.TL;
    const bool real = comp < 3;  // the others: component 0, thread 0 of their column
    if (!real) comp = u = 0;
    const int col = tile * C + l;
    const bool ok = col < a.ncols;
    constexpr unsigned CS = sizeof(cpx<T>);
    const Buf g = buf_of(a.buf);
    const unsigned zs = (unsigned)a.ncols * CS, at = ((unsigned)comp * (unsigned)a.comp_stride + (unsigned)col) * CS;
    cpx<T>* ln = lds + (comp * C + l) * LP;
    constexpr unsigned TS = sizeof(T);
    const Buf K = buf_of(a.kern);
    T kv[kRzProduct][6];
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = idx & (C - 1), kz = idx >> a.csh, col2 = tile * C + l2;
        const int kx = col2 / a.Py;
        int ky = col2 - kx * a.Py;
        const T sy = 2 * ky > a.Py ? (T)-1 : (T)1;
        if (2 * ky > a.Py) ky = a.Py - ky;
        const bool in = 2 * kz <= P && col2 < a.ncols;
        const unsigned ko = ((unsigned)kz * (unsigned)a.k_zs + (unsigned)kx * (unsigned)a.k_xs + (unsigned)ky) * TS;
#pragma unroll
        for (int c = 0; c < 6; ++c) kv[it][c] = buf_ld<T>(K, in ? ko : kBufNone, (unsigned)c * (unsigned)a.k_cs * TS);
        kv[it][1] *= sy;  // mirrored ky: xy and yz odd in y
        kv[it][4] *= sy;
    }
    const int nz = ok ? a.nz : 0;
    rline_fft<T, RM, false, true>(
        s, (const cpx<T>*)a.tws, ln, u, real,
        [&](int e) { return buf_ld<cpx<T>>(g, e < nz ? at + (unsigned)e * zs : kBufNone); },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = idx & (C - 1), kz = idx >> a.csh;
        if (2 * kz <= P && tile * C + l2 < a.ncols) {
            const T(&k)[6] = kv[it];
            cpx<T>* q = lds + l2 * LP;
            tensor_product(q + kz, q + C * LP + kz, q + 2 * C * LP + kz, k);
            if (kz > 0 && 2 * kz < P) {  // the mirrored point: xz and yz odd in z
                const T m[6] = {k[0], k[1], -k[2], k[3], -k[4], k[5]};
                q += P - kz;
                tensor_product(q, q + C * LP, q + 2 * C * LP, m);
            }
        }
    }
    __syncthreads();
    rline_fft<T, RM, true, false>(
        s, (const cpx<T>*)a.tws, ln, u, real, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) { buf_st(g, e < nz ? at + (unsigned)e * zs : kBufNone, conj(x)); });
}

// Along y on one-cell-thick grids: L x bins, three component lines each; spectra xx,
// xy, yy, zz.
template <typename T, int RM>
__device__ inline void body_rky(const RKyArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), L = a.L;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const LaneOf w = rline_lane(s, 3 * L);
    const int comp = w.l / L, l = w.l - comp * L, kx = tile * L + l;
    const bool ok = kx < a.hx;
    constexpr unsigned CS = sizeof(cpx<T>);
    const Buf g = buf_of(a.buf);
    const unsigned at = ((unsigned)comp * (unsigned)a.comp_stride + (unsigned)kx * (unsigned)a.line_stride) * CS;
    cpx<T>* ln = lds + w.l * LP;
    constexpr unsigned TS = sizeof(T);
    const Buf K = buf_of(a.kern);
    const int H1 = P / 2 + 1;
    T kv[kRzProduct][4];
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), ky = idx - l2 * H1, kx2 = tile * L + l2;
        const unsigned ko = ((unsigned)kx2 * (unsigned)a.k_xs + (unsigned)ky) * TS;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            kv[it][c] = buf_ld<T>(K, l2 < L && kx2 < a.hx ? ko : kBufNone, (unsigned)c * (unsigned)a.k_cs * TS);
    }
    const int ny = ok ? a.ny : 0;
    rline_fft<T, RM, false, true>(
        s, (const cpx<T>*)a.tws, ln, w.u, w.real,
        [&](int e) { return buf_ld<cpx<T>>(g, e < ny ? at + (unsigned)e * CS : kBufNone); },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), ky = idx - l2 * H1;
        if (l2 < L && tile * L + l2 < a.hx) {
            cpx<T>* q = lds + l2 * LP;
            const bool mirror = ky > 0 && 2 * ky < P;
            thin_product(q + ky, q + (mirror ? P - ky : ky), mirror, L * LP, kv[it][0], kv[it][1], kv[it][2], kv[it][3]);
        }
    }
    __syncthreads();
    rline_fft<T, RM, true, false>(
        s, (const cpx<T>*)a.tws, ln, w.u, w.real, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) { buf_st(g, e < ny ? at + (unsigned)e * CS : kBufNone, conj(x)); });
}

// Along y on grids two cells thick, the z coupling taken directly (Ky2Args): L x bins,
// six lines each (component, plane).  The frequency pairs a thread takes: L (P / 2 + 1) over
// at least 6 L P / R threads.
constexpr int kRy2Product = 2;

template <typename T, int RM>
__device__ inline void body_rky2(const RKy2Args& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), L = a.L;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const LaneOf w = rline_lane(s, 6 * L);
    const int cz = w.l / L, l = w.l - cz * L, kx = tile * L + l;
    const bool ok = kx < a.hx;
    constexpr unsigned CS = sizeof(cpx<T>);
    const Buf g = buf_of(a.buf);
    const unsigned at = ((unsigned)(cz >> 1) * (unsigned)a.comp_stride + (unsigned)(cz & 1) * (unsigned)a.plane_stride +
                         (unsigned)kx * (unsigned)a.line_stride) * CS;
    cpx<T>* ln = lds + w.l * LP;
    constexpr unsigned TS = sizeof(T);
    const Buf K = buf_of(a.kern);
    const int H1 = P / 2 + 1;
    T kv[kRy2Product][kTwoPlaneTablePlanes];
#pragma unroll
    for (int it = 0; it < kRy2Product; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), ky = idx - l2 * H1, kx2 = tile * L + l2;
        const unsigned ko = ((unsigned)kx2 * (unsigned)a.k_xs + (unsigned)ky) * TS;
#pragma unroll
        for (int c = 0; c < kTwoPlaneTablePlanes; ++c)
            kv[it][c] = buf_ld<T>(K, l2 < L && kx2 < a.hx ? ko : kBufNone, (unsigned)c * (unsigned)a.k_cs * TS);
    }
    const int ny = ok ? a.ny : 0;
    rline_fft<T, RM, false, true>(
        s, (const cpx<T>*)a.tws, ln, w.u, w.real,
        [&](int e) { return buf_ld<cpx<T>>(g, e < ny ? at + (unsigned)e * CS : kBufNone); },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRy2Product; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), ky = idx - l2 * H1;
        if (l2 < L && tile * L + l2 < a.hx) {
            cpx<T>* q = lds + l2 * LP;
            two_plane_product<T>(q + ky, L * LP, (T)1, kv[it]);
            if (ky > 0 && 2 * ky < P) two_plane_product<T>(q + P - ky, L * LP, (T)-1, kv[it]);
        }
    }
    __syncthreads();
    rline_fft<T, RM, true, false>(
        s, (const cpx<T>*)a.tws, ln, w.u, w.real, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) { buf_st(g, e < ny ? at + (unsigned)e * CS : kBufNone, conj(x)); });
}

// ------------------------------------------------------- y, z and k-space in one
// Small 3-D grids: one work-group per x bin holds the bin's plane [3][Pz][Py] in LDS and
// runs the y lines of its nz planes, every z line, the Eq. 14 product and the way back:
// one launch where y forward, z k-space and y inverse are three dependent ones of 4 to 5
// us each at these sizes, and no Py-long spectrum in memory.  Lines are taken in rounds
// of as many as the threads hold.  What bounds it is the chain of LDS stages: bins are
// too few to fill the chip several times over.
constexpr int kRyzChunk = 4;  // product elements a thread loads spectra for at a time

template <typename T, int RM>
__device__ inline void body_ryz(const RYzArgs& a, const LinePlan& ply, const LinePlan& plz, int kx, cpx<T>* lds)
{
    const LineRegs sy(ply), sz(plz);
    const int Py = sy.P, Pz = sz.P, LP = rline_len(Py), PL = Pz * LP;
    const int t = (int)threadIdx.x, NT = blockDim.x, ny = a.ny, nz = a.nz;
    constexpr unsigned CS = sizeof(cpx<T>);
    const Buf g = buf_of((const cpx<T>*)a.buf + (int64_t)kx * a.Sy);
    const T* K = (const T*)a.kern + kx * a.k_xs;
    // Eq. 14 spectra of this thread's elements [ky + Py kz], kRyzChunk of them at a time
    T kv[kRyzChunk][6];
    auto load_k = [&](int i0) {
#pragma unroll
        for (int it = 0; it < kRyzChunk; ++it) {
            const int idx = i0 + t + it * NT;
            int kz = div_by(idx, a.ymul), ky = idx - kz * Py;
            if (2 * ky > Py) ky = Py - ky;
            if (2 * kz > Pz) kz = Pz - kz;
            const T* Kp = K + (idx < Py * Pz ? kz * a.k_zs + ky : 0);
#pragma unroll
            for (int c = 0; c < 6; ++c) kv[it][c] = Kp[c * a.k_cs];
        }
    };
    // the padding planes enter the z lines as zeros
    for (int i = t; i < 3 * (Pz - nz) * LP; i += NT) {
        const int c = i / ((Pz - nz) * LP), r = i - c * (Pz - nz) * LP;
        lds[c * PL + nz * LP + r] = cpx<T>{(T)0, (T)0};
    }
    const int yper = NT / sy.TL, zper = a.zper;
    // y lines: line q = c nz + z, from memory into plane c, row z
    auto y_line = [&](int q0, int& q, bool& real, int& u) {
        const LaneOf w = rline_lane(sy, min(yper, 3 * nz - q0));
        q = q0 + w.l;
        real = w.real;
        u = w.u;
    };
    for (int q0 = 0; q0 < 3 * nz; q0 += yper) {
        int q, u;
        bool real;
        y_line(q0, q, real, u);
        const int c = q / nz, z = q - c * nz;
        const unsigned at = ((unsigned)c * (unsigned)a.comp_stride + (unsigned)z * (unsigned)a.zs) * CS;
        cpx<T>* ln = lds + c * PL + z * LP;
        rline_fft<T, RM, false, true>(
            sy, (const cpx<T>*)a.twsy, ln, u, real,
            [&](int e) { return buf_ld<cpx<T>>(g, e < ny ? at + (unsigned)e * CS : kBufNone); },
            [&](int e, cpx<T> x) { ln[e] = x; });
    }
    load_k(0);
    __syncthreads();
    // z lines: line q = c Py + y, lanes line-fastest (neighbouring entries of a row)
    auto z_lines = [&]() __attribute__((always_inline)) {
        for (int q0 = 0; q0 < 3 * Py; q0 += zper) {
            int u = sz.TL == 1 ? 0 : (zper == 1 ? t : div_by(t, a.zmul));
            int q = q0 + t - u * zper;
            const bool real = u < sz.TL && q < 3 * Py;
            if (!real) u = 0, q = q0;
            const int c = div_by(q, a.ymul);
            cpx<T>* ln = lds + c * PL + (q - c * Py);
            rline_fft<T, RM, true, true, 0>(
                sz, (const cpx<T>*)a.twsz, ln, u, real, [&](int e) { return ln[e * LP]; },
                [&](int e, cpx<T> x) { ln[e * LP] = x; }, LP);
        }
        __syncthreads();
    };
    z_lines();
    for (int i0 = 0; i0 < Py * Pz; i0 += kRyzChunk * NT) {
        if (i0 > 0) load_k(i0);
#pragma unroll
        for (int it = 0; it < kRyzChunk; ++it) {
            const int idx = i0 + t + it * NT;
            if (idx < Py * Pz) {
                // mirrored frequencies: xy odd in y, xz odd in z, yz odd in both
                const int kz = div_by(idx, a.ymul), ky = idx - kz * Py;
                const T my = 2 * ky > Py ? (T)-1 : (T)1, mz = 2 * kz > Pz ? (T)-1 : (T)1;
                const T k[6] = {kv[it][0], my * kv[it][1], mz * kv[it][2], kv[it][3], my * mz * kv[it][4], kv[it][5]};
                cpx<T>* q = lds + kz * LP + ky;
                tensor_product(q, q + PL, q + 2 * PL, k);
            }
        }
    }
    __syncthreads();
    z_lines();
    for (int q0 = 0; q0 < 3 * nz; q0 += yper) {
        int q, u;
        bool real;
        y_line(q0, q, real, u);
        const int c = q / nz, z = q - c * nz;
        const unsigned at = ((unsigned)c * (unsigned)a.comp_stride + (unsigned)z * (unsigned)a.zs) * CS;
        cpx<T>* ln = lds + c * PL + z * LP;
        rline_fft<T, RM, true, false>(
            sy, (const cpx<T>*)a.twsy, ln, u, real, [&](int e) { return ln[e]; },
            [&](int e, cpx<T> x) { buf_st(g, e < ny ? at + (unsigned)e * CS : kBufNone, conj(x)); });
    }
}

}  // namespace mm
