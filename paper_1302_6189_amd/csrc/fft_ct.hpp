// fft_ct.hpp -- 1-D FFTs along contiguous rows whose length is known at
// compile time, alone or fused with the transpose that follows (device code
// of fft_ct.hip).  One instance per 2,3,5-smooth length.
//
// Both kernels are bound by HBM (one read and one write of every point), so
// the work in between is arranged to issue few instructions per point:
//   * L lanes (a power of two) share a row and hold about N / L values each in
//     registers; the Stockham passes exchange them through LDS.  Up to 64 lanes
//     sit in one wave, and the exchanges then need no work-group barrier.
//   * every LDS position is a lane's own base plus a constant: exchange p pads
//     its Stockham blocks (CtPass::PAD values after every Ns R), which keeps
//     writes and reads linear and spreads the lanes over the banks; HBM
//     addresses step by uniform amounts.  A wave of 512-point rows issues 549
//     vector instructions in the fused kernel (710 with computed positions).
//   * the radices, lanes and index arithmetic are constants of the length
//     (ct_choose); radices up to 16 keep most lengths at two or three passes
//     where the run-time-radix unit of fused_generic.hpp takes four or five.
//   * the rows of a group are split at run time over v and over batch slices
//     (CtShape), so short axes fill a group as well as long ones.
#pragma once

#include <hip/hip_runtime.h>

#include "cplx.hpp"
#include "fft_ct_table.hpp"
#include "fft_generic.hpp"
#include "kernels.hpp"
#include "xpose_tile.hpp"

namespace fftrw {

// ---- choice of lanes and radices for a row length ----------------------------
struct CtChoice {
    int L = 0;       // lanes per row
    int np = 0;      // passes
    int pair = 0;    // pass 0 takes two adjacent butterflies per lane (16-byte loads)
    int r[5] = {};   // radices in pass order
    int cost = 1 << 30;
    int rsum = 0;
};

constexpr int kCtRadices[] = {2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16};

constexpr int ct_cdiv(int a, int b) { return (a + b - 1) / b; }
constexpr int ct_mod(int a, int b) { return ((a % b) + b) % b; }

// butterflies per lane of a pass
constexpr int ct_iters(int N, int R, int L, bool pair)
{
    return pair ? 2 * ct_cdiv(N / R / 2, L) : ct_cdiv(N / R, L);
}

constexpr void ct_search(int N, int left, int esz, CtChoice cur, CtChoice &best)
{
    if (left == 1) {
        if (cur.cost < best.cost || (cur.cost == best.cost && cur.rsum < best.rsum)) best = cur;
        return;
    }
    if (cur.np == 5) return;
    for (int R : kCtRadices) {
        // at most 20 complex64 (12 complex128) values per lane, so that four
        // waves per SIMD fit the registers
        if (R > (esz == 8 ? 16 : 10) || left % R) continue;
        const int it = ct_iters(N, R, cur.L, cur.np == 0 && cur.pair);
        if (it * R > (esz == 8 ? 20 : 12) || (cur.np == 0 && cur.pair && (N / R) % 2)) continue;
        CtChoice next = cur;
        next.r[next.np++] = R;
        next.cost += it * R * cur.L * 64 / N + 40;
        next.rsum += R;
        ct_search(N, left / R, esz, next, best);
    }
}

// Lanes and radices of rows of N values of esz bytes: the lowest sum over the
// passes of (work including idle lanes, 64 = none idle) + 40 for the pass's
// exchange; 8-byte instead of 16-byte loads count 16, and lanes beyond what
// leaves a 1024-thread group whole 128-byte runs 24 per halving of the run.
constexpr CtChoice ct_choose(int N, int esz)
{
    CtChoice best;
    for (int L = 1; L <= 256; L *= 2)
        for (int pair = 0; pair <= 1; ++pair) {
            if (pair && (esz != 8 || N % 2 || L * 16 < 128)) continue;
            CtChoice c;
            c.L = L;
            c.pair = pair;
            c.cost = pair || esz != 8 ? 0 : 16;
            const int nt = L <= 16 ? 256 : L <= 32 ? 512 : 1024;
            const int run = nt / L * esz;
            if (run < 128) c.cost += 24 * (128 / run);
            ct_search(N, N, esz, c, best);
        }
    return best;
}

constexpr int ct_max_threads(int L, int esz) { return L * (128 / esz) < 256 ? 256 : L * (128 / esz) > 1024 ? 1024 : L * (128 / esz); }

template <typename C, int N_> struct CtPlan {
    static constexpr int N = N_;
    static constexpr int LINE = 128 / (int)sizeof(C);  // values per 128 bytes
    static constexpr CtChoice c = ct_choose(N_, (int)sizeof(C));
    static constexpr int L = c.L;
    static constexpr int NP = c.np;
    static constexpr int MAXNT = ct_max_threads(L, (int)sizeof(C));
    // rows are read straight into the registers of pass 0 when a row's lanes
    // cover 128 bytes per access, else through LDS
    static constexpr bool DIRECT = L * (int)sizeof(C) * (c.pair ? 2 : 1) >= 128;
    static constexpr bool STORE_DIRECT = L * (int)sizeof(C) >= 128;
    static constexpr bool LAST_PAIR = false;
};

// The same lanes and radices with the first and the last pass's butterflies in
// adjacent pairs per lane, where that leaves no lane idle: rows alone that are
// read and written straight from and to HBM, 16 bytes per lane.
template <typename C, int N_> struct CtStraight : CtPlan<C, N_> {
    using B = CtPlan<C, N_>;
    static constexpr bool pairs(int R)
    {
        return sizeof(C) == 8 && (N_ / R) % 2 == 0 && ct_iters(N_, R, B::L, true) == ct_iters(N_, R, B::L, false);
    }
    static constexpr CtChoice paired()
    {
        CtChoice p = B::c;
        p.pair = pairs(p.r[0]);
        return p;
    }
    static constexpr CtChoice c = paired();
    static constexpr bool LAST_PAIR = pairs(B::c.r[B::NP - 1]);
    static constexpr bool DIRECT = true, STORE_DIRECT = true;
};

// compile-time description of pass p of a plan, and of the exchange after it
template <class P, int p> struct CtPass {
    static constexpr int R = P::c.r[p];
    static constexpr int Ns = CtPass<P, p - 1>::Ns * CtPass<P, p - 1>::R;
    static constexpr int NB = P::N / R;
    static constexpr bool PAIR = p == P::NP - 1 && P::LAST_PAIR;
    static constexpr int IT = ct_iters(P::N, R, P::L, PAIR);
    // (pass 0 has no twiddles)
    static constexpr int tw_off =
        p == 1 ? 0 : CtPass<P, p - 1>::tw_off + CtPass<P, p - 1>::Ns * (CtPass<P, p - 1>::R - 1);
    // The lanes of a write come in runs of Ns neighbours, one run per block of
    // Ns R values: the padded block length is congruent to Ns modulo a line,
    // so that consecutive runs fall on consecutive banks (odd for Ns past a
    // line, where any spread will do).
    static constexpr int BLK = Ns * R;
    static constexpr int PAD = Ns >= P::LINE ? 0 : ct_mod(Ns - BLK, P::LINE);
};
template <class P> struct CtPass<P, 0> {
    static constexpr int R = P::c.r[0];
    static constexpr int Ns = 1;
    static constexpr int NB = P::N / R;
    static constexpr bool PAIR = P::c.pair != 0;
    static constexpr int IT = ct_iters(P::N, R, P::L, PAIR);
    static constexpr int tw_off = 0;
    static constexpr int BLK = R;
    static constexpr int PAD = 1 - R % 2;  // lanes a block apart: odd
};

template <class P, int p> constexpr int ct_max_span()
{
    // extent of a row's exchange buffer over the exchanges 0 .. p - 1
    if constexpr (p == 0) {
        return P::N;
    } else {
        using S = CtPass<P, p - 1>;
        constexpr int here = P::N + S::PAD * (P::N / S::BLK - 1), before = ct_max_span<P, p - 1>();
        return here > before ? here : before;
    }
}
// LDS pitch of the rows' exchange buffers: odd, so that rows start on different banks
template <class P> constexpr int ct_row_pitch() { return ct_max_span<P, P::NP - 1>() | 1; }

// bases of batch slice g (innermost batch axis first) in A and B
__device__ __forceinline__ void ct_slice(const XposeDesc &d, const CtShape &s, uint32_t g, int64_t *ab, int64_t *bb)
{
    int64_t a = 0, b = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        // (axes past nbat have size 0 and strides 0, and g is 0 by then)
        const uint32_t q = s.db[i](g);
        const int c = (int)(g - q * (uint32_t)d.bsize[i]);
        g = q;
        a += c * d.ba[i];
        b += c * d.bb[i];
    }
    *ab = a;
    *bb = b;
}

// butterfly m of a lane, and whether every lane has one
template <class P, int p> __device__ __forceinline__ int ct_j(int lane, int m)
{
    return CtPass<P, p>::PAIR ? 2 * (lane + (m >> 1) * P::L) + (m & 1) : lane + m * P::L;
}
template <class P, int p> constexpr bool ct_all(int m)
{
    return CtPass<P, p>::PAIR ? ((m >> 1) + 1) * 2 * P::L <= CtPass<P, p>::NB : (m + 1) * P::L <= CtPass<P, p>::NB;
}

// values and twiddles of one lane in pass p
template <class P, int p, typename C> struct CtVals {
    C x[CtPass<P, p>::IT * CtPass<P, p>::R];
};
template <class P, int p, typename C> struct CtTw {
    C t[p > 0 ? CtPass<P, p>::IT * (CtPass<P, p>::R - 1) : 1];
};

struct CtNoTw {};
template <class P, int p, typename C, bool in = (p < P::NP)> struct CtTwOf { using type = CtNoTw; };
template <class P, int p, typename C> struct CtTwOf<P, p, C, true> { using type = CtTw<P, p, C>; };
template <class P, int p, typename C> using CtTwNext = typename CtTwOf<P, p, C>::type;

// Twiddles of pass p, w_{Ns R}^{i k} at [i - 1][k]: consecutive lanes read
// consecutive entries.  They depend on the lane only and are loaded ahead of
// the pass.
template <class P, int p, typename C>
__device__ __forceinline__ void ct_load_tw(CtTw<P, p, C> &w, int lane, const C *__restrict__ tw)
{
    using S = CtPass<P, p>;
    if constexpr (p > 0) {
#pragma unroll
        for (int m = 0; m < S::IT; ++m) {
            const uint32_t k = (uint32_t)ct_j<P, p>(lane, m) % S::Ns;
#pragma unroll
            for (int i = 1; i < S::R; ++i) w.t[m * (S::R - 1) + i - 1] = (tw + S::tw_off + (i - 1) * S::Ns)[k];
        }
    }
}

template <class P, int p, typename C>
__device__ __forceinline__ void ct_butterflies(CtVals<P, p, C> &v, const CtTw<P, p, C> &w)
{
    using S = CtPass<P, p>;
#pragma unroll
    for (int m = 0; m < S::IT; ++m) {
        if constexpr (p > 0) {
#pragma unroll
            for (int i = 1; i < S::R; ++i) v.x[m * S::R + i] = cmul(v.x[m * S::R + i], w.t[m * (S::R - 1) + i - 1]);
        }
        Dft<S::R, -1, C>::run(v.x + m * S::R);
    }
}

// pass p's inputs from the row's LDS buffer: element e at e + PAD (e / BLK) of
// the exchange before it (elements as loaded for pass 0); BLK divides NB, so
// the inputs of a butterfly sit a constant apart
template <class P, int p, typename C>
__device__ __forceinline__ void ct_read_row(CtVals<P, p, C> &v, const C *row, int lane)
{
    using S = CtPass<P, p>;
    constexpr int BLK = p > 0 ? CtPass<P, p - (p > 0)>::BLK : P::N;
    constexpr int PAD = p > 0 ? CtPass<P, p - (p > 0)>::PAD : 0;
    constexpr int STEP = p > 0 ? S::NB + PAD * (S::NB / BLK) : S::NB;
#pragma unroll
    for (int m = 0; m < S::IT; ++m) {
        const int j = ct_j<P, p>(lane, m);
        if (ct_all<P, p>(m) || j < S::NB) {
            const C *q = row + (PAD ? j + PAD * (int)((uint32_t)j / BLK) : j);
#pragma unroll
            for (int i = 0; i < S::R; ++i) v.x[m * S::R + i] = q[i * STEP];
        }
    }
}

// pass p's outputs to the row's LDS buffer (Stockham positions, padded)
template <class P, int p, typename C>
__device__ __forceinline__ void ct_write_row(const CtVals<P, p, C> &v, C *row, int lane)
{
    using S = CtPass<P, p>;
#pragma unroll
    for (int m = 0; m < S::IT; ++m) {
        const int j = ct_j<P, p>(lane, m);
        if (ct_all<P, p>(m) || j < S::NB) {
            const int b = (uint32_t)j / S::Ns, k = j - b * S::Ns;
            C *q = row + b * (S::BLK + S::PAD) + k;
#pragma unroll
            for (int i = 0; i < S::R; ++i) q[i * S::Ns] = v.x[m * S::R + i];
        }
    }
}

// Passes p.. of the lane's values; w are pass p's twiddles and wn pass p + 1's
// (loaded by the caller: pass 1's go out with the rows, so that both arrive in
// one memory round trip).  The last pass's outputs are handed to fin.
template <class P, int p, typename C, typename Fin>
__device__ __forceinline__ void ct_passes(CtVals<P, p, C> &v, const CtTw<P, p, C> &w, const CtTwNext<P, p + 1, C> &wn,
                                          C *row, int lane, const C *__restrict__ tw, Fin &&fin)
{
    ct_butterflies<P, p, C>(v, w);
    if constexpr (p + 1 < P::NP) {
        CtTwNext<P, p + 2, C> wnn;
        if constexpr (p + 2 < P::NP) ct_load_tw<P, p + 2, C>(wnn, lane, tw);
        CtVals<P, p + 1, C> vn;
        ct_write_row<P, p, C>(v, row, lane);
        row_sync(P::L <= 64);
        ct_read_row<P, p + 1, C>(vn, row, lane);
        if constexpr (p + 2 < P::NP) row_sync(P::L <= 64);
        ct_passes<P, p + 1, C>(vn, wn, wnn, row, lane, tw, fin);
    } else {
        fin(v);
    }
}

template <typename C> struct CtRaw;
template <> struct CtRaw<float2> { using type = xf2; };
template <> struct CtRaw<double2> { using type = xd2; };

// One HBM access, streaming (non-temporal) or cached.
template <bool NT, typename T> __device__ __forceinline__ T ct_ld(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    return *p;
}
template <bool NT, typename T> __device__ __forceinline__ void ct_st(T v, T *p)
{
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// pass 0's inputs straight from the row in HBM
template <class P, bool NT, typename C>
__device__ __forceinline__ void ct_load_direct(CtVals<P, 0, C> &v, const C *src, int lane)
{
    using S = CtPass<P, 0>;
    using V = typename CtRaw<C>::type;
    if constexpr (S::PAIR) {
#pragma unroll
        for (int m = 0; m < S::IT; m += 2) {
            const int j = ct_j<P, 0>(lane, m);
            if (ct_all<P, 0>(m) || j < S::NB) {
#pragma unroll
                for (int i = 0; i < S::R; ++i) {
                    const xf4 q = ct_ld<NT>(reinterpret_cast<const xf4 *>(src + j + i * S::NB));
                    v.x[m * S::R + i] = mk<C>(q.x, q.y);
                    v.x[(m + 1) * S::R + i] = mk<C>(q.z, q.w);
                }
            }
        }
    } else {
#pragma unroll
        for (int m = 0; m < S::IT; ++m) {
            const int j = ct_j<P, 0>(lane, m);
            if (ct_all<P, 0>(m) || j < S::NB) {
#pragma unroll
                for (int i = 0; i < S::R; ++i) {
                    const V q = ct_ld<NT>(reinterpret_cast<const V *>(src + j + i * S::NB));
                    v.x[m * S::R + i] = mk<C>(q.x, q.y);
                }
            }
        }
    }
}

template <class P, int p, typename C> __device__ __forceinline__ void ct_conj(CtVals<P, p, C> &v)
{
    using S = CtPass<P, p>;
#pragma unroll
    for (int e = 0; e < S::IT * S::R; ++e) v.x[e].y = -v.x[e].y;
}

constexpr int ct_log2ceil(int n)
{
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

// Short rows between HBM and their LDS buffers: 2^LW threads share a row, W
// neighbouring values each, and step over the rows by a uniform amount.
template <class P, typename C> struct CtStage {
    static constexpr int W = sizeof(C) == 8 && P::N % 2 == 0 ? 2 : 1;
    static constexpr int NW = P::N / W;
    static constexpr int LW = ct_log2ceil(NW);
    static constexpr int IT = ct_cdiv(1 << LW, P::L);
};

// rows to LDS: row rho starts at src + rho step, or at src + rowa[rho] (rowa
// not null); all loads are issued before the first LDS store
template <class P, bool NT, typename C>
__device__ __forceinline__ void ct_load_staged(C *lds, const C *src, int64_t step, const int64_t *rowa, int nth,
                                               int nrows)
{
    using S = CtStage<P, C>;
    using V = typename CtRaw<C>::type;
    constexpr int RP = ct_row_pitch<P>();
    const int c = (threadIdx.x & ((1 << S::LW) - 1)) * S::W;
    const int rho0 = threadIdx.x >> S::LW, drho = nth >> S::LW;
    C val[S::IT][S::W];
    const C *p = src + c + (rowa ? 0 : rho0 * step);
    const int64_t dp = drho * step;
#pragma unroll
    for (int it = 0; it < S::IT; ++it) {
        const int rho = rho0 + it * drho;
        if (rho < nrows && c < P::N) {
            const C *q = rowa ? src + c + rowa[rho] : p;
            if constexpr (S::W == 2) {
                const xf4 w = ct_ld<NT>(reinterpret_cast<const xf4 *>(q));
                val[it][0] = mk<C>(w.x, w.y);
                val[it][1] = mk<C>(w.z, w.w);
            } else {
                const V w = ct_ld<NT>(reinterpret_cast<const V *>(q));
                val[it][0] = mk<C>(w.x, w.y);
            }
        }
        p += dp;
    }
    C *l = lds + rho0 * RP + c;
#pragma unroll
    for (int it = 0; it < S::IT; ++it) {
        if (rho0 + it * drho < nrows && c < P::N) {
#pragma unroll
            for (int w = 0; w < S::W; ++w) l[w] = val[it][w];
        }
        l += drho * RP;
    }
}

// rows from LDS to HBM, row rho at dst + rho N
template <class P, bool NT, typename C>
__device__ __forceinline__ void ct_store_staged(C *dst, const C *lds, int nth, int nrows)
{
    using S = CtStage<P, C>;
    using V = typename CtRaw<C>::type;
    constexpr int RP = ct_row_pitch<P>();
    const int c = (threadIdx.x & ((1 << S::LW) - 1)) * S::W;
    const int rho0 = threadIdx.x >> S::LW, drho = nth >> S::LW;
    C *p = dst + c + (int64_t)rho0 * P::N;
    const C *l = lds + rho0 * RP + c;
#pragma unroll
    for (int it = 0; it < S::IT; ++it) {
        if (rho0 + it * drho < nrows && c < P::N) {
            if constexpr (S::W == 2)
                ct_st<NT>(xf4{l[0].x, l[0].y, l[1].x, l[1].y}, reinterpret_cast<xf4 *>(p));
            else
                ct_st<NT>(V{l[0].x, l[0].y}, reinterpret_cast<V *>(p));
        }
        p += drho * P::N;
        l += drho * RP;
    }
}

// Rows alone that are not whole 128-byte lines, between HBM and their LDS
// buffers as one block, which all threads copy from end to end, so that an
// access covers whole lines but at the block's ends.
template <class P, typename C> struct CtBlock {
    static constexpr int W = sizeof(C) == 8 ? 2 : 1;
    static constexpr int IT = ct_cdiv(ct_cdiv(P::N, W), P::L);
    static constexpr int SKIP = ct_row_pitch<P>() - P::N;  // LDS positions between rows

    // f(it, e, l, l2, n): the it-th access of this thread is of the block's
    // values e .. e + n - 1, which sit at l and (W = 2) l2 in LDS
    template <typename F> static __device__ __forceinline__ void each(int nth, int nrows, F &&f)
    {
        const int total = nrows * P::N;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int e = (threadIdx.x + it * nth) * W;
            if (e >= total) continue;
            const int row = (uint32_t)e / P::N, l = e + SKIP * row;
            // (a pair of an odd row's last value and the next row's first)
            const int l2 = l + 1 + (P::N % 2 != 0 && SKIP != 0 && e + 1 == (row + 1) * P::N ? SKIP : 0);
            f(it, e, l, l2, P::N % 2 != 0 ? min(W, total - e) : W);
        }
    }

    template <bool NT> static __device__ __forceinline__ void load(C *lds, const C *src, int nth, int nrows)
    {
        using V = typename CtRaw<C>::type;
        C val[IT][W];
        each(nth, nrows, [&](int it, int e, int, int, int n) {
            if constexpr (W == 2) {
                if (n == 2) {
                    const xf4 w = ct_ld<NT>(reinterpret_cast<const xf4 *>(src + e));
                    val[it][0] = mk<C>(w.x, w.y);
                    val[it][1] = mk<C>(w.z, w.w);
                    return;
                }
            }
            const V w = ct_ld<NT>(reinterpret_cast<const V *>(src + e));
            val[it][0] = mk<C>(w.x, w.y);
        });
        each(nth, nrows, [&](int it, int, int l, int l2, int n) {
            lds[l] = val[it][0];
            if constexpr (W == 2)
                if (n == 2) lds[l2] = val[it][1];
        });
    }

    template <bool NT> static __device__ __forceinline__ void store(C *dst, const C *lds, int nth, int nrows)
    {
        using V = typename CtRaw<C>::type;
        each(nth, nrows, [&](int, int e, int l, int l2, int n) {
            if constexpr (W == 2) {
                if (n == 2) {
                    ct_st<NT>(xf4{lds[l].x, lds[l].y, lds[l2].x, lds[l2].y}, reinterpret_cast<xf4 *>(dst + e));
                    return;
                }
            }
            ct_st<NT>(V{lds[l].x, lds[l].y}, reinterpret_cast<V *>(dst + e));
        });
    }
};

// position of column (row of the group) `col` in a frequency's line of the
// output block: one value of padding per 128 bytes
template <typename C> __device__ __forceinline__ int ct_col(int col) { return col + (col >> (sizeof(C) == 8 ? 4 : 3)); }

// The fused kernel's results, frequency k of row rho at k sp + ct_col(rho) in
// LDS, to layout B: frequency k of row (gi, r) at bbase(gi) + k b_su + v0 + r,
// W consecutive v per access.
template <class P, bool NT, int W, typename C>
__device__ __forceinline__ void ct_store_runs(C *out, const C *lds, const CtShape &s, int64_t b_su,
                                              const int64_t *bbase, int64_t bbase0, int64_t v0, int nv, int ng)
{
    constexpr int N = P::N, IT = ct_cdiv(N, P::L * W);
    using V = typename CtRaw<C>::type;
    const int nth = P::L << s.lr;
    auto value = [](const C *l) {
        if constexpr (W == 2)
            return xf4{l[0].x, l[0].y, l[1].x, l[1].y};
        else
            return V{l[0].x, l[0].y};
    };
    using T = decltype(value(lds));
    T q[IT];
    if (s.G == 1) {
        // one slice: the threads of a power of two share a frequency's run and
        // step over the frequencies by a uniform amount
        const int lw = s.lr - (W == 2 ? 1 : 0);
        const int k0 = threadIdx.x >> lw, dk = nth >> lw;
        const int r = (threadIdx.x & ((1 << lw) - 1)) * W;
        const C *l = lds + k0 * s.sp + ct_col<C>(r);
        C *p = out + bbase0 + v0 + r + k0 * b_su;
        const int64_t dp = dk * b_su;
        if (r >= nv) return;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if (N % (P::L * W) == 0 || k0 + it * dk < N) q[it] = value(l);
            l += dk * s.sp;
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if (N % (P::L * W) == 0 || k0 + it * dk < N) ct_st<NT>(q[it], reinterpret_cast<T *>(p));
            p += dp;
        }
        return;
    }
    // several slices: e = (gi N + k) nvw + r / W; division by nvw = nv / W
    // through its rounded-up reciprocal, exact for e < 2^16 (its error adds
    // less than e / 2^32 < 1 / nvw to e / nvw)
    const int nvw = nv / W;
    const uint32_t mg = 0xffffffffu / (uint32_t)nvw + 1u;
    const int total = ng * N * nvw;
    auto split = [&](int e, int &gi, int &k, int &r) {
        const int row = nvw == 1 ? e : (int)__umulhi((uint32_t)e, mg);
        gi = (uint32_t)row / N;
        k = row - gi * N;
        r = (e - row * nvw) * W;
    };
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int e = threadIdx.x + it * nth;
        int gi, k, r;
        split(e, gi, k, r);
        if (e < total) {
            const int col = gi * s.rw + r;
            // (with pairs rw is even: a pair shares its 128 bytes)
            q[it] = value(lds + k * s.sp + ct_col<C>(col));
        }
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const int e = threadIdx.x + it * nth;
        int gi, k, r;
        split(e, gi, k, r);
        if (e < total) ct_st<NT>(q[it], reinterpret_cast<T *>(out + bbase[gi] + k * b_su + v0 + r));
    }
}

// ---- FFT step fused with the transpose that follows it -----------------------
// A work-group transforms rw rows along u (the last axis of layout A),
// consecutive in v (the last axis of layout B), in each of G batch slices, and
// writes layout B through an LDS block: every k of a slice becomes one run of
// consecutive v.  The first ncount groups of the launch count the transpose's
// owner changes instead (count_share).
template <typename C, int N>
__global__ void __launch_bounds__((CtPlan<C, N>::MAXNT))
    ct_fused_kernel(const void *in_, void *out_, const XposeDesc d, const CtShape s, const void *tw_, double scale,
                    int ncount)
{
    using P = CtPlan<C, N>;
    extern __shared__ __align__(16) unsigned char smem[];
    if (blockIdx.x < (unsigned)ncount) {
        count_share(d, blockIdx.x, ncount, reinterpret_cast<unsigned long long *>(smem));
        return;
    }
    C *lds = reinterpret_cast<C *>(smem);
    int64_t *bbase = reinterpret_cast<int64_t *>(smem + s.tab);
    int64_t *rowa = bbase + s.G;  // first element of every row (short rows)
    const C *in = reinterpret_cast<const C *>(in_);
    C *out = reinterpret_cast<C *>(out_);
    const C *__restrict__ tw = reinterpret_cast<const C *>(tw_);
    const int nth = P::L << s.lr;

    uint32_t unit = blockIdx.x - (unsigned)ncount;
    if (s.per_xcd) {
        // work-groups go to the 8 XCDs in turn; neighbouring units share the
        // cache lines at the ends of their runs
        unit = (unit & 7) * s.per_xcd + (unit >> 3);
        if (unit >= s.units) return;
    }
    const uint32_t tg = s.dtv(unit);
    const int v0 = (int)(unit - tg * s.tiles_v) * s.rw;
    const uint32_t g0 = tg * s.G;
    const int nv = min(s.rw, (int)d.Nv - v0);
    const int ng = min(s.G, (int)(d.nslices - g0));
    int64_t abase0 = 0, bbase0 = 0;
    if (s.G == 1) ct_slice(d, s, g0, &abase0, &bbase0);

    const int rho = threadIdx.x / P::L, lane = threadIdx.x % P::L;
    CtVals<P, 0, C> v;
    CtTw<P, 0, C> w0;
    CtTwNext<P, 1, C> w1;
    if constexpr (P::NP > 1) ct_load_tw<P, 1, C>(w1, lane, tw);
    C *row = lds + rho * ct_row_pitch<P>();
    if constexpr (P::DIRECT) {
        int gi = 0, r = rho;
        int64_t ab = abase0;
        if (s.G > 1) {
            gi = rho / s.rw;
            r = rho - gi * s.rw;
            int64_t bb;
            if (gi < ng) {
                ct_slice(d, s, g0 + gi, &ab, &bb);
                if (r == 0 && lane == 0) bbase[gi] = bb;
            }
        }
        if (gi < ng && r < nv) {
            const C *src = in + ab + (v0 + r) * d.a_sv;
            either(s.nt_load, [&](auto nt) { ct_load_direct<P, nt.value, C>(v, src, lane); });
        } else {
#pragma unroll
            for (int e = 0; e < CtPass<P, 0>::IT * CtPass<P, 0>::R; ++e) v.x[e] = mk<C>(0, 0);
        }
    } else {
        // rows packed (gi nv + r), their bases in LDS
        const int nrows = ng * nv;
        if (s.G > 1) {
            if ((int)threadIdx.x < nrows) {
                const int gi = threadIdx.x / (uint32_t)nv, r = threadIdx.x - gi * nv;
                int64_t ab, bb;
                ct_slice(d, s, g0 + gi, &ab, &bb);
                rowa[threadIdx.x] = ab + (v0 + r) * d.a_sv;
                if (r == 0) bbase[gi] = bb;
            }
            __syncthreads();
        }
        const C *src = s.G > 1 ? in : in + abase0 + (int64_t)v0 * d.a_sv;
        const int64_t *tab = s.G > 1 ? rowa : nullptr;
        either(s.nt_load, [&](auto nt) { ct_load_staged<P, nt.value, C>(lds, src, d.a_sv, tab, nth, nrows); });
    }
    if constexpr (!P::DIRECT) {
        __syncthreads();
        // (rows past the last read what the buffer holds; nothing is stored
        // for them)
        ct_read_row<P, 0, C>(v, row, lane);
        if constexpr (P::NP > 1) row_sync(P::L <= 64);
    }
    if (s.inverse) ct_conj<P, 0, C>(v);
    ct_passes<P, 0, C>(v, w0, w1, row, lane, tw, [&](CtVals<P, P::NP - 1, C> &y) {
        using S = CtPass<P, P::NP - 1>;
        __syncthreads();  // every row's last reads are done
        if (s.inverse) ct_conj<P, P::NP - 1, C>(y);
        if (s.do_scale) {
            const typename RealOf<C>::type sx = (typename RealOf<C>::type)scale;
#pragma unroll
            for (int e = 0; e < S::IT * S::R; ++e) y.x[e] = cscale(y.x[e], sx);
        }
        // row rho's column of the block; packed rows (short rows) sit at
        // gi rw + r like the others
        int col = rho;
        if constexpr (!P::DIRECT)
            if (nv != s.rw) {
                const int gi = rho / (uint32_t)nv;
                col = gi * s.rw + (rho - gi * nv);
            }
        if (col < (1 << s.lr)) {
            C *l = lds + ct_col<C>(col);
#pragma unroll
            for (int m = 0; m < S::IT; ++m) {
                const int j = ct_j<P, P::NP - 1>(lane, m);
                if (ct_all<P, P::NP - 1>(m) || j < S::NB) {
                    C *q = l + j * s.sp;
#pragma unroll
                    for (int i = 0; i < S::R; ++i) {
                        *q = y.x[m * S::R + i];
                        q += S::NB * s.sp;
                    }
                }
            }
        }
    });
    __syncthreads();
    // two values per 16-byte store when N_v and rw are even: every stride of
    // layout B other than v's is then even, so each pair starts 16 bytes
    // aligned
    if constexpr (sizeof(C) == 8) {
        if (((d.Nv | s.rw) & 1) == 0 && s.lr > 0) {
            either(s.nt_store, [&](auto nt) {
                ct_store_runs<P, nt.value, 2, C>(out, lds, s, d.b_su, bbase, bbase0, v0, nv, ng);
            });
            return;
        }
    }
    either(s.nt_store, [&](auto nt) {
        ct_store_runs<P, nt.value, 1, C>(out, lds, s, d.b_su, bbase, bbase0, v0, nv, ng);
    });
}

// ---- FFT step alone: rows in place or from `in` to `out` ----------------------
// P: CtPlan or CtStraight.  BLOCK: the group's rows go through LDS as one block
// (CtBlock); otherwise row by row, as the plan says.
template <typename C, class P, bool BLOCK>
__global__ void __launch_bounds__(P::MAXNT)
    ct_rows_kernel(const void *in_, void *out_, int64_t nrows, const void *tw_, double scale, const CtRowsShape s)
{
    constexpr int N = P::N;
    using B = CtBlock<P, C>;
    constexpr bool DIRECT = P::DIRECT && !BLOCK, STORE_DIRECT = P::STORE_DIRECT && !BLOCK;
    extern __shared__ __align__(16) unsigned char smem[];
    C *lds = reinterpret_cast<C *>(smem);
    const int64_t row0 = (int64_t)blockIdx.x << s.lr;
    const C *in = reinterpret_cast<const C *>(in_) + row0 * N;
    C *out = reinterpret_cast<C *>(out_) + row0 * N;
    const C *__restrict__ tw = reinterpret_cast<const C *>(tw_);
    const int nth = P::L << s.lr;
    const int here = (int)min<int64_t>((int64_t)1 << s.lr, nrows - row0);
    const int rho = threadIdx.x / P::L, lane = threadIdx.x % P::L;
    C *row = lds + rho * ct_row_pitch<P>();
    CtVals<P, 0, C> v;
    CtTw<P, 0, C> w0;
    CtTwNext<P, 1, C> w1;
    if constexpr (P::NP > 1) ct_load_tw<P, 1, C>(w1, lane, tw);
    if constexpr (DIRECT) {
        if (rho < here) {
            either(s.flags & kCtNtLoad, [&](auto nt) { ct_load_direct<P, nt.value, C>(v, in + rho * N, lane); });
        } else {
#pragma unroll
            for (int e = 0; e < CtPass<P, 0>::IT * CtPass<P, 0>::R; ++e) v.x[e] = mk<C>(0, 0);
        }
    } else {
        either(s.flags & kCtNtLoad, [&](auto nt) {
            if constexpr (BLOCK)
                B::template load<nt.value>(lds, in, nth, here);
            else
                ct_load_staged<P, nt.value, C>(lds, in, N, nullptr, nth, here);
        });
        __syncthreads();
        ct_read_row<P, 0, C>(v, row, lane);
        row_sync(P::L <= 64);
    }
    if (s.flags & kCtInverse) ct_conj<P, 0, C>(v);
    ct_passes<P, 0, C>(v, w0, w1, row, lane, tw, [&](CtVals<P, P::NP - 1, C> &y) {
        using S = CtPass<P, P::NP - 1>;
        using V = typename CtRaw<C>::type;
        if constexpr (!STORE_DIRECT && P::NP > 1) row_sync(P::L <= 64);
        if (s.flags & kCtInverse) ct_conj<P, P::NP - 1, C>(y);
        if (s.flags & kCtScale) {
            const typename RealOf<C>::type sx = (typename RealOf<C>::type)scale;
#pragma unroll
            for (int e = 0; e < S::IT * S::R; ++e) y.x[e] = cscale(y.x[e], sx);
        }
        if constexpr (STORE_DIRECT && S::PAIR) {
#pragma unroll
            for (int m = 0; m < S::IT; m += 2) {
                const int j = ct_j<P, P::NP - 1>(lane, m);
                if (rho < here && (ct_all<P, P::NP - 1>(m) || j < S::NB)) {
                    xf4 *p = reinterpret_cast<xf4 *>(out + rho * N + j);
                    either(s.flags & kCtNtStore, [&](auto nt) {
#pragma unroll
                        for (int i = 0; i < S::R; ++i) {
                            C a = y.x[m * S::R + i], b = y.x[(m + 1) * S::R + i];
                            // (values, not loads of two neighbours of y, which
                            // would keep y in scratch memory)
                            asm("" : "+v"(a.x), "+v"(a.y), "+v"(b.x), "+v"(b.y));
                            ct_st<nt.value>(xf4{a.x, a.y, b.x, b.y}, p + i * (S::NB / 2));
                        }
                    });
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m < S::IT; ++m) {
                const int j = ct_j<P, P::NP - 1>(lane, m);
                if (ct_all<P, P::NP - 1>(m) || j < S::NB) {
                    if constexpr (STORE_DIRECT) {
                        if (rho < here) {
                            V *p = reinterpret_cast<V *>(out + rho * N + j);
                            either(s.flags & kCtNtStore, [&](auto nt) {
#pragma unroll
                                for (int i = 0; i < S::R; ++i)
                                    ct_st<nt.value>(V{y.x[m * S::R + i].x, y.x[m * S::R + i].y}, p + i * S::NB);
                            });
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < S::R; ++i) row[j + i * S::NB] = y.x[m * S::R + i];
                    }
                }
            }
        }
    });
    if constexpr (!STORE_DIRECT) {
        __syncthreads();
        either(s.flags & kCtNtStore, [&](auto nt) {
            if constexpr (BLOCK)
                B::template store<nt.value>(out, lds, nth, here);
            else
                ct_store_staged<P, nt.value, C>(out, lds, nth, here);
        });
    }
}

}  // namespace fftrw
