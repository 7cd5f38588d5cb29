// mm_rline.hpp -- FFT passes of any 7-smooth padded length, with the length a
// runtime value and the transforms in registers.
//
// A line of P points is worked by TL = P / (its smallest radix) threads, one
// butterfly per thread and stage: the radices of a LinePlan (2 .. 16, composites
// such as 6, 10, 12, 14 and 15 included, so lengths up to 256 take two stages and up
// to 4096 mostly three) are chosen on the host, and each stage switches on its radix
// (the same for the whole work-group) to a body unrolled for it.  The first stage
// takes its inputs straight from where they are (global memory, or LDS for an inverse
// after the k-space product), the stages between exchange through LDS, and the last
// one hands its outputs to the caller.  Every index is linear in the stage's loop
// variable (one addition an element, no division inside a stage), and the twiddles of
// a stage lie [r][k] so that consecutive threads read consecutive entries.
//
// What these replace ran every length through one LDS-staged body with 16 elements a
// thread: a division and a remainder per element to find its line, 215 to 233
// registers (two waves a SIMD) and strided twiddle reads.
//
// Spectrum layout: as everywhere, S = [3][nz][hx][Sy].
#pragma once
#include "mm_fast.hpp"
#include "mm_kernels.hpp"

namespace mm {

// ------------------------------------------------------- composite register DFTs
// Coprime factors by the prime-factor map (no twiddles): with N = A B,
// n = (B n1 + A n2) mod N, k = (B b k1 + A a k2) mod N, B b = 1 mod A, A a = 1 mod B.
constexpr int inv_mod(int x, int m)
{
    for (int i = 1; i < m; ++i)
        if (x * i % m == 1) return i;
    return 1;
}

template <typename T, int A, int B>
__device__ inline void dft_pfa(cpx<T>* v)
{
    constexpr int N = A * B;
    cpx<T> a[B][A];
#pragma unroll
    for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
        for (int n1 = 0; n1 < A; ++n1) a[n2][n1] = v[(B * n1 + A * n2) % N];
        Dft<T, A>::run(a[n2]);
    }
    constexpr int e1 = B * inv_mod(B % A, A), e2 = A * inv_mod(A % B, B);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) {
        cpx<T> b[B];
#pragma unroll
        for (int n2 = 0; n2 < B; ++n2) b[n2] = a[n2][k1];
        Dft<T, B>::run(b);
#pragma unroll
        for (int k2 = 0; k2 < B; ++k2) v[(e1 * k1 + e2 * k2) % N] = b[k2];
    }
}

template <typename T>
struct Dft<T, 6> {
    __device__ static inline void run(cpx<T>* v) { dft_pfa<T, 2, 3>(v); }
};
template <typename T>
struct Dft<T, 10> {
    __device__ static inline void run(cpx<T>* v) { dft_pfa<T, 2, 5>(v); }
};
template <typename T>
struct Dft<T, 12> {
    __device__ static inline void run(cpx<T>* v) { dft_pfa<T, 4, 3>(v); }
};
template <typename T>
struct Dft<T, 14> {
    __device__ static inline void run(cpx<T>* v) { dft_pfa<T, 2, 7>(v); }
};
template <typename T>
struct Dft<T, 15> {
    __device__ static inline void run(cpx<T>* v) { dft_pfa<T, 3, 5>(v); }
};
// 9 = 3 x 3 with the twiddles exp(-2 pi i n2 k1 / 9)
template <typename T>
struct Dft<T, 9> {
    __device__ static inline void run(cpx<T>* v)
    {
        const cpx<T> w1 = {(T)0.76604444311897803520, (T)-0.64278760968653932632};
        const cpx<T> w2 = {(T)0.17364817766693034885, (T)-0.98480775301220805937};
        const cpx<T> w4 = {(T)-0.93969262078590838405, (T)-0.34202014332566873304};
        cpx<T> a[3][3];
#pragma unroll
        for (int n2 = 0; n2 < 3; ++n2) {
#pragma unroll
            for (int n1 = 0; n1 < 3; ++n1) a[n2][n1] = v[3 * n1 + n2];
            Dft<T, 3>::run(a[n2]);
        }
        a[1][1] = cmul(a[1][1], w1);
        a[1][2] = cmul(a[1][2], w2);
        a[2][1] = cmul(a[2][1], w2);
        a[2][2] = cmul(a[2][2], w4);
#pragma unroll
        for (int k1 = 0; k1 < 3; ++k1) {
            cpx<T> b[3] = {a[0][k1], a[1][k1], a[2][k1]};
            Dft<T, 3>::run(b);
#pragma unroll
            for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = b[k2];
        }
    }
};

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
    LineStage st[kMaxLineStages];
    __device__ inline explicit LineRegs(const LinePlan& s)
        : P(sgpr(s.P)), ns(sgpr(s.ns)), TL(sgpr(s.TL)), tmul((unsigned)sgpr((int)s.tmul))
    {
#pragma unroll
        for (int q = 0; q < kMaxLineStages; ++q)
            st[q] = LineStage{sgpr(s.R[q]), sgpr(s.p[q]), sgpr(s.m[q]), sgpr(s.toff[q]), (unsigned)sgpr((int)s.pmul[q])};
    }
    __device__ inline LineStage stage(int q) const
    {
        static_assert(kMaxLineStages == 5, "stages picked by hand");
        // by value through readfirstlane: a choice between the fields' addresses would
        // put the schedule into private memory
        auto pick = [q](int a1, int a2, int a3, int a4) {
            a1 = sgpr(a1), a2 = sgpr(a2), a3 = sgpr(a3), a4 = sgpr(a4);
            return q == 1 ? a1 : (q == 2 ? a2 : (q == 3 ? a3 : a4));
        };
        return LineStage{pick(st[1].R, st[2].R, st[3].R, st[4].R), pick(st[1].p, st[2].p, st[3].p, st[4].p),
                         pick(st[1].m, st[2].m, st[3].m, st[4].m),
                         pick(st[1].toff, st[2].toff, st[3].toff, st[4].toff),
                         (unsigned)pick((int)st[1].pmul, (int)st[2].pmul, (int)st[3].pmul, (int)st[4].pmul)};
    }
};

// The radices a kernel serves: all, or (RM = 10) those up to 10, whose butterflies need
// about 40 registers fewer.
#define MM_RADIX_CASES(X)                                         \
    X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)                 \
    X(12) X(14) X(15) X(16)

// Forward FFT of one line by its TL threads (u = this thread's number in the line;
// act = false: a thread that only joins the barriers).  get(e) delivers input e of the
// first stage (it is called by every thread, with e below P, and must not branch),
// put(e, value) takes output e.  SYNC: the inputs come from LDS that the stages
// overwrite, so every thread's reads end before the first write.
// tws: the line's stage twiddles (LinePlan::toff).
//
// The switches hold nothing but loads and arithmetic on one array v shared by their
// cases: with a divergent branch or a barrier inside, the compiler keeps every case's
// values alive side by side (256 registers and hundreds spilled).
template <typename T, int RM, bool SYNC, class Get, class Put>
__device__ inline void rline_fft(const LineRegs& s, const cpx<T>* __restrict__ tws, cpx<T>* ln, int u, bool act,
                                 Get get, Put put)
{
    const int ns = s.ns;
    cpx<T> v[RM];
    {
        const int m = s.st[0].m, R = s.st[0].R;
        const bool on = act && u < m;
        const int i = on ? u : 0;
        switch (R) {
#define X(RR)                                                                   \
    case RR:                                                                    \
        if constexpr (RR <= RM) {                                               \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) v[r] = get(i + r * m); \
            Dft<T, RR>::run(v);                                                 \
        }                                                                       \
        break;
            MM_RADIX_CASES(X)
#undef X
        default: break;
        }
        if (SYNC) __syncthreads();
        if (ns == 1) {
            if (on) {
#pragma unroll
                for (int r = 0; r < RM; ++r)
                    if (r < R) put(r, v[r]);
            }
            return;
        }
        if (on) {
            cpx<T>* o = ln + u * R;
#pragma unroll
            for (int r = 0; r < RM; ++r)
                if (r < R) o[r] = v[r];
        }
        __syncthreads();
    }
    for (int q = 1; q < ns; ++q) {
        const LineStage c = s.stage(q);
        const int m = c.m, p = c.p;
        const bool on = act && u < m;
        const int i = on ? u : 0;
        // the last stage has p = m, so its k is i and its outputs sit where its inputs were
        const bool last = q == ns - 1;
        const int k = last ? i : i - div_by(i, c.pmul) * p;
        const cpx<T>* w = tws + c.toff;
        switch (c.R) {
#define X(RR)                                                                            \
    case RR:                                                                             \
        if constexpr (RR <= RM) {                                                        \
            cpx<T> tw[RR];                                                               \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) tw[r] = w[(r - 1) * p + k];   \
            _Pragma("unroll") for (int r = 0; r < RR; ++r) v[r] = ln[i + r * m];         \
            _Pragma("unroll") for (int r = 1; r < RR; ++r) v[r] = cmul(v[r], tw[r]);     \
            Dft<T, RR>::run(v);                                                          \
        }                                                                                \
        break;
            MM_RADIX_CASES(X)
#undef X
        default: break;
        }
        if (last) {
            if (on) {
#pragma unroll
                for (int r = 0; r < RM; ++r)
                    if (r < c.R) put(i + r * m, v[r]);
            }
            return;
        }
        __syncthreads();
        if (on) {
            cpx<T>* o = ln + (i - k) * c.R + k;
#pragma unroll
            for (int r = 0; r < RM; ++r)
                if (r < c.R) o[r * p] = v[r];
        }
        __syncthreads();
    }
}

// This thread's line (of `per` lines side by side) and its number in it.
struct LaneOf {
    int l, u;
};
__device__ inline LaneOf rline_lane(const LineRegs& s)
{
    const int t = (int)threadIdx.x;
    const int l = s.TL == 1 ? t : div_by(t, s.tmul);
    return LaneOf{l, t - l * s.TL};
}

// ------------------------------------------------------------------ y lines
template <typename T, int RM, bool INV>
__device__ inline void body_ryline(const RYArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const LaneOf w = rline_lane(s);
    const int line = tile * a.L + w.l;
    const bool ok = w.l < a.L && line < a.nlines;
    int mline = ok ? line : 0;
    if (a.kx_major) mline = (mline % a.kx_major) * (a.nlines / a.kx_major) + mline / a.kx_major;
    cpx<T>* g = (cpx<T>*)a.buf + (int64_t)mline * a.line_stride;
    const int nin = a.nin, nout = a.nout;
    rline_fft<T, RM, false>(
        s, (const cpx<T>*)a.tws, lds + (ok ? w.l : 0) * rline_len(s.P), w.u, ok,
        [&](int e) {
            const cpx<T> x = g[e < nin ? e : 0];
            return e < nin ? (INV ? conj(x) : x) : cpx<T>{(T)0, (T)0};
        },
        [&](int e, cpx<T> v) {
            if (e < nout) g[e] = INV ? conj(v) : v;
        });
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
    const LaneOf w = rline_lane(s);
    const int y0 = yb + 2 * w.l;
    const bool act = w.l < L;
    const bool ok0 = act && y0 < a.ny, ok1 = act && y0 + 1 < a.ny;
    const T* in = (const T*)a.in + ((int64_t)plane * a.ny + (ok0 ? y0 : 0)) * a.nx;
    const T* in1 = in + (ok1 ? a.nx : 0);
    cpx<T>* ln = lds + (act ? w.l : 0) * LP;
    const int nx = a.nx;
    rline_fft<T, RM, false>(
        s, (const cpx<T>*)a.tws, ln, w.u, act,
        [&](int e) {
            const int i = e < nx ? e : 0;
            const T re = in[i], im = in1[i];
            return cpx<T>{e < nx && ok0 ? re : (T)0, e < nx && ok1 ? im : (T)0};
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
    const LaneOf w = rline_lane(s);
    const bool act = w.l < L;
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
    const cpx<T>* ra = lds + (act ? 2 * w.l : 0) * hx;
    const cpx<T>* rb = ra + hx;
    const int y0 = yb + 2 * w.l, nx = a.nx;
    const bool ok0 = y0 < a.ny, ok1 = y0 + 1 < a.ny;
    T* out = (T*)a.out + ((int64_t)plane * a.ny + y0) * nx;
    rline_fft<T, RM, true>(
        s, (const cpx<T>*)a.tws, lds + (act ? w.l : 0) * LP, w.u, act,
        [&](int k) {
            const bool lo = k < hx;
            cpx<T> A = ra[lo ? k : P - k], B = rb[lo ? k : P - k];
            if (k == 0 || 2 * k == P) A.im = B.im = (T)0;  // DC and Nyquist bins of a real row are real
            // conj(A + i B) below hx, conj(conj A + i conj B) above: inverse by conjugation
            return lo ? cpx<T>{A.re - B.im, -A.im - B.re} : cpx<T>{A.re + B.im, A.im - B.re};
        },
        [&](int e, cpx<T> v) {  // result a + i b = conj(v)
            if (e < nx) {
                if (ok0) out[e] = v.re;
                if (ok1) out[nx + e] = -v.im;
            }
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

// Product elements a thread takes: C P of them over at least 3 C P / R threads, R <= 16.
constexpr int kRzProduct = 6;

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
    const int comp = s.TL == 1 ? v : div_by(v, s.tmul), u = v - comp * s.TL;
    const int col = tile * C + l;
    const bool act = comp < 3, ok = act && col < a.ncols;
    const int64_t zs = a.ncols;
    cpx<T>* g = (cpx<T>*)a.buf + (ok ? comp * a.comp_stride + col : 0);
    cpx<T>* ln = lds + ((act ? comp : 0) * C + l) * LP;
    const T* K = (const T*)a.kern;
    T kv[kRzProduct][6];
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = idx & (C - 1), e = idx >> a.csh, col2 = tile * C + l2;
#pragma unroll
        for (int c = 0; c < 6; ++c) kv[it][c] = (T)0;
        if (e < P && col2 < a.ncols) {
            const int kx = col2 / a.Py;
            int ky = col2 - kx * a.Py, kz = e;
            const bool my = 2 * ky > a.Py, mz = 2 * kz > P;
            if (my) ky = a.Py - ky;
            if (mz) kz = P - kz;
            const T* Kp = K + kz * a.k_zs + kx * a.k_xs + ky;
#pragma unroll
            for (int c = 0; c < 6; ++c) kv[it][c] = Kp[c * a.k_cs];
        }
    }
    const int nz = a.nz;
    rline_fft<T, RM, false>(
        s, (const cpx<T>*)a.tws, ln, u, act,
        [&](int e) {
            const bool in = ok && e < nz;
            const cpx<T> x = g[in ? e * zs : 0];
            return in ? x : cpx<T>{(T)0, (T)0};
        },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = idx & (C - 1), e = idx >> a.csh, col2 = tile * C + l2;
        if (e < P && col2 < a.ncols) {
            // mirrored frequencies: xy odd in y, xz odd in z, yz odd in both
            const int kx = col2 / a.Py, ky = col2 - kx * a.Py;
            const T sy = 2 * ky > a.Py ? (T)-1 : (T)1, sz = 2 * e > P ? (T)-1 : (T)1;
            const T k[6] = {kv[it][0], sy * kv[it][1], sz * kv[it][2], kv[it][3], sy * sz * kv[it][4], kv[it][5]};
            cpx<T>* q = lds + l2 * LP + e;
            tensor_product(q, q + C * LP, q + 2 * C * LP, k);
        }
    }
    __syncthreads();
    rline_fft<T, RM, true>(
        s, (const cpx<T>*)a.tws, ln, u, act, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) {
            if (ok && e < nz) g[e * zs] = conj(x);
        });
}

// Along y on one-cell-thick grids: L x bins, three component lines each; spectra xx,
// xy, yy, zz.
template <typename T, int RM>
__device__ inline void body_rky(const RKyArgs& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), L = a.L;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const LaneOf w = rline_lane(s);
    const int comp = w.l / L, l = w.l - comp * L, kx = tile * L + l;
    const bool act = comp < 3, ok = act && kx < a.hx;
    cpx<T>* g = (cpx<T>*)a.buf + (ok ? comp * a.comp_stride + (int64_t)kx * a.line_stride : 0);
    cpx<T>* ln = lds + (act ? w.l : 0) * LP;
    const T* K = (const T*)a.kern;
    T kv[kRzProduct][4];
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), e = idx - l2 * P, kx2 = tile * L + l2;
#pragma unroll
        for (int c = 0; c < 4; ++c) kv[it][c] = (T)0;
        if (l2 < L && kx2 < a.hx) {
            const T* Kp = K + (int64_t)kx2 * a.k_xs + (2 * e > P ? P - e : e);
#pragma unroll
            for (int c = 0; c < 4; ++c) kv[it][c] = Kp[c * a.k_cs];
        }
    }
    const int ny = a.ny;
    rline_fft<T, RM, false>(
        s, (const cpx<T>*)a.tws, ln, w.u, act,
        [&](int e) {
            const bool in = ok && e < ny;
            const cpx<T> x = g[in ? e : 0];
            return in ? x : cpx<T>{(T)0, (T)0};
        },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRzProduct; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), e = idx - l2 * P;
        if (l2 < L && tile * L + l2 < a.hx) {
            const T sy = 2 * e > P ? (T)-1 : (T)1;
            cpx<T>* qx = lds + l2 * LP + e;
            cpx<T>*qy = qx + L * LP, *qz = qy + L * LP;
            const cpx<T> mx = *qx, my = *qy, mz = *qz;
            const T kxx = kv[it][0], kxy = sy * kv[it][1], kyy = kv[it][2], kzz = kv[it][3];
            *qx = conj(cpx<T>{kxx * mx.re + kxy * my.re, kxx * mx.im + kxy * my.im});
            *qy = conj(cpx<T>{kxy * mx.re + kyy * my.re, kxy * mx.im + kyy * my.im});
            *qz = conj(cpx<T>{kzz * mz.re, kzz * mz.im});
        }
    }
    __syncthreads();
    rline_fft<T, RM, true>(
        s, (const cpx<T>*)a.tws, ln, w.u, act, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) {
            if (ok && e < ny) g[e] = conj(x);
        });
}

// Along y on grids two cells thick, the z coupling taken directly (Ky2Args): L x bins,
// six lines each (component, plane).  The product elements a thread takes: L P over at
// least 6 L P / R threads.
constexpr int kRy2Product = 3;

template <typename T, int RM>
__device__ inline void body_rky2(const RKy2Args& a, const LinePlan& pl, int tile, cpx<T>* lds)
{
    const LineRegs s(pl);
    const int P = s.P, LP = rline_len(P), L = a.L;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const LaneOf w = rline_lane(s);
    const int cz = w.l / L, l = w.l - cz * L, kx = tile * L + l;
    const bool act = cz < 6, ok = act && kx < a.hx;
    cpx<T>* g = (cpx<T>*)a.buf + (ok ? (cz >> 1) * a.comp_stride + (cz & 1) * a.plane_stride + (int64_t)kx * a.line_stride : 0);
    cpx<T>* ln = lds + (act ? w.l : 0) * LP;
    const T* K = (const T*)a.kern;
    T kv[kRy2Product][kTwoPlaneTablePlanes];
#pragma unroll
    for (int it = 0; it < kRy2Product; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), e = idx - l2 * P, kx2 = tile * L + l2;
        const bool in = l2 < L && kx2 < a.hx;
        const T* Kp = K + (in ? (int64_t)kx2 * a.k_xs + (2 * e > P ? P - e : e) : 0);
#pragma unroll
        for (int c = 0; c < kTwoPlaneTablePlanes; ++c) kv[it][c] = Kp[c * a.k_cs];
    }
    const int ny = a.ny;
    rline_fft<T, RM, false>(
        s, (const cpx<T>*)a.tws, ln, w.u, act,
        [&](int e) {
            const bool in = ok && e < ny;
            const cpx<T> x = g[in ? e : 0];
            return in ? x : cpx<T>{(T)0, (T)0};
        },
        [&](int e, cpx<T> x) { ln[e] = x; });
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kRy2Product; ++it) {
        const int idx = t + it * NT;
        const int l2 = div_by(idx, a.dmul), e = idx - l2 * P;
        if (l2 < L && tile * L + l2 < a.hx) two_plane_product<T>(lds + l2 * LP + e, L * LP, 2 * e > P ? (T)-1 : (T)1, kv[it]);
    }
    __syncthreads();
    rline_fft<T, RM, true>(
        s, (const cpx<T>*)a.tws, ln, w.u, act, [&](int e) { return ln[e]; },
        [&](int e, cpx<T> x) {
            if (ok && e < ny) g[e] = conj(x);
        });
}

}  // namespace mm
