// mm_rfused.hpp -- the fused stage pass and the fused adjoint stage (mm_fused.hpp) for
// any 7-smooth x length: the same steps with the transforms of mm_rline.hpp.
#pragma once
#include "mm_fused.hpp"
#include "mm_rline.hpp"

namespace mm {

// The gather takes the 2 L rows of three components, hx bins each: at most kRfGather
// loads a thread in flight.
constexpr int kRfGather = 8;

// As fused_block, with L row pairs of length s.P; cell rows of w = nx + 1 values, the last
// one a slot for what is cut off (it reads as the zero padding of the forward transform).
// Component region of LDS: rfused_region entries.
template <typename T, int RM, class Pre, class Update>
__device__ inline void rfused_block(const RFusedArgs& g, const LineRegs& s, int tile, bool fwd, cpx<T>* lds, T* cell,
                                    Pre pre, Update update)
{
    const int P = s.P, LP = rline_len(P), hx = P / 2 + 1, L = g.L, rows = 2 * L, nx = g.nx, ny = g.ny, W = nx + 1;
    const int reg = rfused_region(L, P);
    const int tpp = (ny + rows - 1) / rows;
    const int z = tile / tpp, yb = (tile - z * tpp) * rows;
    const int t = (int)threadIdx.x, NT = blockDim.x;
    const LaneOf w = rline_lane(s, 3 * L);
    const int comp = w.l / L, l = w.l - comp * L;
    cpx<T>* base = lds + comp * reg;
    constexpr unsigned CS = sizeof(cpx<T>);

    // ---- x inverse: element idx = (c hx + kx) rows + rr of the block, all loads of a
    // round issued before its LDS stores
    {
        const Buf in = buf_of(g.S_in);
        const int nel = 3 * hx * rows;
        for (int i0 = 0; i0 < nel; i0 += kRfGather * NT) {
            cpx<T> gv[kRfGather];
#pragma unroll
            for (int it = 0; it < kRfGather; ++it) {
                const int idx = i0 + t + it * NT;
                const int b = idx >> g.rsh, rr = idx - (b << g.rsh);  // rows = 1 << rsh
                const int c = div_by(b, g.hmul), kx = b - c * hx, y = yb + rr;
                const unsigned at = ((unsigned)((c * g.nz + z) * hx + kx) * (unsigned)g.sy + (unsigned)y) * CS;
                gv[it] = buf_ld<cpx<T>>(in, idx < nel && y < ny ? at : kBufNone);
            }
            if (i0 == 0) pre();
#pragma unroll
            for (int it = 0; it < kRfGather; ++it) {
                const int idx = i0 + t + it * NT;
                const int b = idx >> g.rsh, rr = idx - (b << g.rsh);
                const int c = div_by(b, g.hmul), kx = b - c * hx;
                if (idx < nel) lds[c * reg + rr * hx + kx] = gv[it];
            }
        }
    }
    __syncthreads();
    {
        const cpx<T>* ra = base + (2 * l) * hx;
        const cpx<T>* rb = ra + hx;
        T* cl = cell + (comp * rows + 2 * l) * W;
        rline_fft<T, RM, true, true>(
            s, (const cpx<T>*)g.tws, base + l * LP, w.u, w.real,
            [&](int k) {
                const bool lo = k < hx;
                cpx<T> A = ra[lo ? k : P - k], B = rb[lo ? k : P - k];
                if (k == 0 || 2 * k == P) A.im = B.im = (T)0;  // DC and Nyquist bins of a real row are real
                return lo ? cpx<T>{A.re - B.im, -A.im - B.re} : cpx<T>{A.re + B.im, A.im - B.re};
            },
            [&](int e, cpx<T> v) {  // rows 2l, 2l + 1 of the block: re, -im
                const int i = e < nx ? e : nx;
                cl[i] = v.re;
                cl[W + i] = -v.im;
            });
    }
    __syncthreads();

    update(z, yb);
    if (!fwd) return;
    for (int r = t; r < 3 * rows; r += NT) cell[r * W + nx] = (T)0;
    __syncthreads();

    // ---- x forward of the block's new rows, half spectrum stored transposed
    {
        const T* cl = cell + (comp * rows + 2 * l) * W;
        const bool ok0 = yb + 2 * l < ny, ok1 = yb + 2 * l + 1 < ny;
        rline_fft<T, RM, true, true>(
            s, (const cpx<T>*)g.tws, base + l * LP, w.u, w.real,
            [&](int e) {
                const int i = e < nx ? e : nx;
                const T re = cl[i], im = cl[W + i];
                return cpx<T>{ok0 ? re : (T)0, ok1 ? im : (T)0};
            },
            [&](int e, cpx<T> v) { base[l * LP + e] = v; });
    }
    __syncthreads();
    cpx<T>* out = (cpx<T>*)g.S_out;
    for (int idx = t; idx < 3 * hx * L; idx += NT) {
        const int b = idx >> (g.rsh - 1), q = idx - (b << (g.rsh - 1));
        const int c = div_by(b, g.hmul), kx = b - c * hx;
        const cpx<T>* lq = lds + c * reg + q * LP;
        const cpx<T> zk = lq[kx], zm = lq[kx == 0 ? 0 : P - kx];
        // Z = FFT(a + i b): A = (Z_k + conj Z_-k)/2, B = (Z_k - conj Z_-k)/(2i)
        const cpx<T> A = scale(zk + conj(zm), (T)0.5);
        const cpx<T> B = scale(mul_mi(zk - conj(zm)), (T)0.5);
        const int y = yb + 2 * q;
        cpx<T>* o = out + ((int64_t)(c * g.nz + z) * hx + kx) * g.sy + y;
        if (y < ny) o[0] = A;
        if (y + 1 < ny) o[1] = B;
    }
}

// PRE > 0: a thread has at most PRE cells, and their loads go out with the gather's (see
// body_fused_stage); 0: three cells' loads at a time before their updates.
template <typename T, int RM, int PRE>
__device__ inline void body_rfused_stage(const FusedStageArgs<T>& f, const RFusedArgs& g, const LinePlan& pl, int tile,
                                         cpx<T>* lds, T* cell)
{
    constexpr int CH = PRE > 0 ? PRE : 3;
    const LineRegs s(pl);
    const LlgArgs<T>& a = f.g;
    const int rows = 2 * g.L, tpp = (a.ny + rows - 1) / rows, tid = (int)threadIdx.x;
    const int z0 = tile / tpp;
    const CellBlock b{z0, (tile - z0 * tpp) * rows, rows, a.nx + 1, (int)blockDim.x};
    const int nc = PRE > 0 ? PRE : (rows * a.nx + b.nt - 1) / b.nt;
    StageIn<T, CH> in;
    auto update = [&](int, int) {
        for (int q0 = 0; q0 < nc; q0 += CH) {
            if (PRE == 0) in.load(a, b, tid, q0, nc);
            in.update(a, b, tid, q0, nc, cell, f.hout);
        }
    };
    auto pre = [&] {
        if constexpr (PRE > 0) in.load(a, b, tid, 0, nc);
    };
    rfused_block<T, RM>(g, s, tile, true, lds, cell, pre, update);
}

template <typename T, int RM>
__device__ inline void body_rfused_adjoint(const FusedAdjArgs<T>& f, const RFusedArgs& g, const LinePlan& pl, int tile,
                                           cpx<T>* lds, T* cell)
{
    const LineRegs s(pl);
    const int rows = 2 * g.L, nt = blockDim.x, nc = (rows * f.a.nx + nt - 1) / nt;
    auto update = [&](int z, int yb) {
        fused_adjoint_cells(f, CellBlock{z, yb, rows, f.a.nx + 1, nt}, (int)threadIdx.x, nc, cell);
    };
    rfused_block<T, RM>(g, s, tile, f.mode != 0, lds, cell, [] {}, update);
}

}  // namespace mm
