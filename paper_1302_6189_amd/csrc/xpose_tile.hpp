// xpose_tile.hpp -- one tile of the transpose between two decompositions
// (device code shared by the stand-alone kernel and the persistent batched
// kernel).
//
// The array moves from layout A (decomposition pi_t) to layout B (pi_{t+1}).
// Consecutive decompositions always have different last axes, so the
// permutation is a tiled 2-D transpose between u (fastest axis of A) and v
// (fastest axis of B), batched over the other M-2 axes.  A work-group reads a
// TU x TV tile (times G batch slices) along u, transposes it through LDS and
// writes it along v, so both sides are coalesced; with an even u (v) size a
// thread moves two neighbouring values per 16-byte access.
//
// Owner counting: virtual process p owns a contiguous range of rows over the
// first k axes of its decomposition (Eqs. (13)-(15)).  Below level M the
// first k axes of A never include u and those of B never include v, so along
// a (slice, v) row A's owner is fixed and B's row index grows linearly with u:
// the points that keep their owner are the u whose B row falls in that
// owner's range, an interval.  At level M (more processes than rows, the last
// case of Eq. (13)) the row index is the point's whole linear index, so A's
// owner also grows with u (and B's row index also depends on v); the row then
// splits into pieces of constant A owner, each counted the same way (row_keep).
// The rest of the row moves.  Summed over tiles this is the paper's
// communication amount for the transpose.
#pragma once

#include <hip/hip_runtime.h>

#include "cplx.hpp"
#include "kernels.hpp"

namespace fftrw {

constexpr int kMaxG = 256;
constexpr int kTileBatch = 8;  // rows a thread loads (or stores) before it waits

typedef float xf4 __attribute__((ext_vector_type(4)));
typedef float xf2 __attribute__((ext_vector_type(2)));
typedef double xd2 __attribute__((ext_vector_type(2)));

template <bool NT = true, typename C> __device__ __forceinline__ C xld(const C *p)
{
    if constexpr (!NT) {
        return gld(p);
    } else if constexpr (sizeof(C) == 8) {
        xf2 w = gld_nt(reinterpret_cast<const xf2 *>(p));
        return mk<C>(w.x, w.y);
    } else {
        xd2 w = gld_nt(reinterpret_cast<const xd2 *>(p));
        return mk<C>(w.x, w.y);
    }
}
template <bool NT = true, typename C> __device__ __forceinline__ void xst(C *p, C v)
{
    using V = typename std::conditional<sizeof(C) == 8, xf2, xd2>::type;
    const V w = {v.x, v.y};
    if constexpr (NT)
        gst_nt(w, reinterpret_cast<V *>(p));
    else
        gst(w, reinterpret_cast<V *>(p));
}

__device__ __forceinline__ int64_t owner_of_row(int64_t r, int64_t P, int64_t R, bool narrow)
{
    if (narrow) return (int64_t)(((uint32_t)(r + 1) * (uint32_t)P - 1u) / (uint32_t)R);
    return ((r + 1) * P - 1) / R;
}

// coordinates of batch slice s (innermost batch axis first) and its bases;
// plans keep the slice count below 2^31 (sizes are at most 4096), so 32-bit
// divisions suffice
__device__ __forceinline__ void slice_coords(const XposeDesc &d, int64_t s, int *c, int64_t *ab, int64_t *bb)
{
    int64_t a = 0, b = 0;
    uint32_t su = (uint32_t)s;
    for (int i = 0; i < d.nbat; ++i) {
        const uint32_t n = (uint32_t)d.bsize[i];
        const uint32_t q = su / n;
        const uint32_t ci = su - q * n;
        su = q;
        c[i] = (int)ci;
        a += (int64_t)ci * d.ba[i];
        b += (int64_t)ci * d.bb[i];
    }
    *ab = a;
    *bb = b;
}

// Row indices of a batch slice's points in A and B, affine in u and v: A's
// grows with u only at level M, B's with v only there.
struct SliceRows {
    int64_t ra0 = 0, wau = 0, wav = 0;
    int64_t rb0 = 0, wbu = 0, wbv = 0;
};

__device__ __forceinline__ SliceRows slice_rows(const XposeDesc &d, const int *c)
{
    SliceRows r;
    for (int j = 0; j < d.ka; ++j) {
        const int src = d.srca[j];
        if (src == 4)
            r.wau = d.wa[j];
        else if (src == 3)
            r.wav = d.wa[j];
        else
            r.ra0 += (int64_t)c[src] * d.wa[j];
    }
    for (int j = 0; j < d.kb; ++j) {
        const int src = d.srcb[j];
        if (src == 4)
            r.wbu = d.wb[j];
        else if (src == 3)
            r.wbv = d.wb[j];
        else
            r.rb0 += (int64_t)c[src] * d.wb[j];
    }
    return r;
}

// floor(x / y) for x >= 0, y > 0, and ceil(x / w) for w > 0.  When R P < 2^32
// for both layouts (narrow) every operand is under 2^32, so 32-bit divisions
// suffice.
__device__ __forceinline__ int64_t owner_fdiv(int64_t x, int64_t y, bool narrow)
{
    return narrow ? (int64_t)((uint32_t)x / (uint32_t)y) : x / y;
}
__device__ __forceinline__ int64_t owner_cdiv(int64_t x, int64_t w, bool narrow)
{
    if (x < 0) return -owner_fdiv(-x, w, narrow);
    const int64_t q = owner_fdiv(x, w, narrow);
    return q + (q * w != x ? 1 : 0);
}

// u in [a, b) whose row rb0 + u wbu of B lies in the range of process o
__device__ __forceinline__ int64_t keep_in_b(const XposeDesc &d, int64_t rb0, int64_t wbu, int64_t o, int64_t a,
                                             int64_t b)
{
    const bool narrow = d.owner32 != 0;
    if (wbu == 0) return owner_of_row(rb0, d.P, d.Rb, narrow) == o ? b - a : 0;
    const int64_t lo = owner_fdiv(d.Rb * o, d.P, narrow) - rb0, hi = owner_fdiv(d.Rb * (o + 1), d.P, narrow) - rb0;
    const int64_t k0 = max<int64_t>(a, owner_cdiv(lo, wbu, narrow)), k1 = min<int64_t>(b, owner_cdiv(hi, wbu, narrow));
    return max<int64_t>(0, k1 - k0);
}

// Points of the row (batch coordinates c, v) with u in [u0, u0 + nu) that keep
// their owner.  Owners are monotone in the row index, so the row is a
// sequence of pieces of constant A owner o, and inside a piece the u whose B
// row lies in o's range form an interval.
__device__ __forceinline__ int64_t row_keep(const XposeDesc &d, const SliceRows &r, int64_t v, int64_t u0, int64_t nu)
{
    const bool narrow = d.owner32 != 0;
    const int64_t ra0 = r.ra0 + v * r.wav, rb0 = r.rb0 + v * r.wbv;
    if (r.wau == 0) {
        int64_t o = owner_of_row(ra0, d.P, d.Ra, narrow);
        if (d.mu) o = d.mu[o];
        return keep_in_b(d, rb0, r.wbu, o, u0, u0 + nu);
    }
    int64_t keep = 0;
    for (int64_t u = u0, end = u0 + nu; u < end;) {
        const int64_t oa = owner_of_row(ra0 + u * r.wau, d.P, d.Ra, narrow);
        // first u past this piece: A row reaches the start of range oa + 1
        const int64_t next =
            min<int64_t>(end, owner_cdiv(owner_fdiv(d.Ra * (oa + 1), d.P, narrow) - ra0, r.wau, narrow));
        keep += keep_in_b(d, rb0, r.wbu, d.mu ? (int64_t)d.mu[oa] : oa, u, next);
        u = next;
    }
    return keep;
}

// Points of the rows v in [v0, v1) of a batch slice that keep their owner,
// below level M: A's owner is constant along u and B's along v, so the rows
// come in pieces of constant A owner whose intervals of u are the same.
__device__ __forceinline__ int64_t rows_keep(const XposeDesc &d, const int *c, int64_t v0, int64_t v1)
{
    const bool narrow = d.owner32 != 0;
    const SliceRows r = slice_rows(d, c);
    int64_t keep = 0;
    for (int64_t v = v0; v < v1;) {
        const int64_t oa = owner_of_row(r.ra0 + v * r.wav, d.P, d.Ra, narrow);
        int64_t next = v1;
        if (r.wav != 0)
            next = min<int64_t>(v1, owner_cdiv(owner_fdiv(d.Ra * (oa + 1), d.P, narrow) - r.ra0, r.wav, narrow));
        keep += (next - v) * keep_in_b(d, r.rb0, r.wbu, d.mu ? (int64_t)d.mu[oa] : oa, 0, d.Nu);
        v = next;
    }
    return keep;
}

// Points of one tile whose owner changes, this thread's share (one (slice, v)
// row at a time).
__device__ __forceinline__ int tile_moved(const XposeDesc &d, int64_t g0, int ng, int64_t u0, int nu, int64_t v0,
                                          int nv)
{
    int moved = 0;
    for (int i = threadIdx.x; i < ng * nv; i += kThreads) {
        const int g = i / nv, iv = i - g * nv;
        int c[3];
        int64_t ab, bb;
        slice_coords(d, g0 + g, c, &ab, &bb);
        moved += nu - (int)row_keep(d, slice_rows(d, c), v0 + iv, u0, nu);
    }
    return moved;
}

// Owner changes of a whole transpose, counted by `groups` work-groups.  The
// count depends on the decompositions alone: on groups of their own it costs
// the transform nothing (512^3: 1.2% when the row groups counted in front of
// their first barrier), and short kernels no reset launch (32^3 complex128
// 18.9 -> 13.8 us), as every word of the counter is written.
//
// Whole rows: the items are slices, or parts of slices when there are few.
__host__ __device__ inline uint32_t count_chunks(const XposeDesc &d)
{
    const uint32_t n = d.nslices < 8192 ? 8192u / (uint32_t)d.nslices : 1u;
    return n < (uint32_t)d.Nv ? n : (uint32_t)d.Nv;
}
// Split rows (level M): an item is one row's share of 2^lg parts along u, lg
// being count - 2.  A row comes in about count_pieces pieces of constant A
// owner, of seven 64-bit divisions each.
inline int64_t count_pieces(const XposeDesc &d)
{
    for (int j = 0; j < d.ka; ++j)
        if (d.srca[j] == 4) return (int64_t)((__int128)d.P * d.Nu / d.Ra) + 1;
    return 1;
}
// whole rows: two items a thread; split rows: one
inline int count_groups(const XposeDesc &d, int threads)
{
    const int64_t n = d.count >= 2 ? ((d.nslices * d.Nv) << (d.count - 2)) / threads
                                   : d.nslices * count_chunks(d) / (2 * threads);
    return (int)(n < 16 ? 16 : n > kCountBlock ? kCountBlock : (n + 7) / 8 * 8);
}

// The share of group `group`; `part` holds one word per wave.
__device__ __forceinline__ void count_share(const XposeDesc &d, int group, int groups, unsigned long long *part)
{
    const uint64_t first = (uint64_t)group * blockDim.x + threadIdx.x, step = (uint64_t)groups * blockDim.x;
    unsigned long long moved = 0;
    int c[3];
    int64_t ab, bb;
    if (d.count >= 2) {
        const int lg = d.count - 2;
        const uint64_t rows = (uint64_t)(d.nslices * d.Nv);
        const int64_t len = (d.Nu + (1 << lg) - 1) >> lg;
        for (uint64_t i = first; i < rows << lg; i += step) {
            const uint64_t row = i >> lg;
            const int64_t u0 = (int64_t)(i & ((1u << lg) - 1)) * len, nu = min<int64_t>(len, d.Nu - u0);
            if (nu <= 0) continue;
            const uint64_t g = rows >> 32 ? row / (uint32_t)d.Nv : (uint32_t)row / (uint32_t)d.Nv;
            slice_coords(d, (int64_t)g, c, &ab, &bb);
            moved += (unsigned long long)(nu - row_keep(d, slice_rows(d, c), (int64_t)(row - g * d.Nv), u0, nu));
        }
    } else {
        const uint32_t Nv = (uint32_t)d.Nv, ns = (uint32_t)d.nslices, chunks = count_chunks(d);
        const uint32_t per = (Nv + chunks - 1) / chunks;
        for (uint64_t i = first; i < (uint64_t)ns * chunks; i += step) {
            // (chunks > 1 only below 8192 slices: 32 bits hold the product)
            const uint32_t g = chunks == 1 ? (uint32_t)i : (uint32_t)i / chunks;
            const uint32_t v0 = ((uint32_t)i - g * chunks) * per, v1 = min(Nv, v0 + per);
            if (v0 >= v1) continue;
            slice_coords(d, g, c, &ab, &bb);
            moved += (unsigned long long)((int64_t)(v1 - v0) * d.Nu - rows_keep(d, c, v0, v1));
        }
    }
    for (int off = 32; off > 0; off >>= 1) moved += __shfl_xor(moved, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = moved;
    __syncthreads();
    if (threadIdx.x == 0)
        for (unsigned w = 1; w < blockDim.x / 64; ++w) moved += part[w];
    // the group's word, and zeros to the other words of its residue
    for (int w = group + threadIdx.x * groups; w < kCountBlock; w += blockDim.x * groups)
        d.counter[w] = w == group ? moved : 0;
}

// LDS bytes of a tile, 16-byte aligned; launchers reserve 16 more bytes
// after it (xpose_tile writes the loads of items past the tile there)
__host__ __device__ inline size_t xpose_tile_bytes(const XposeDesc &d, size_t esz)
{
    size_t b = (size_t)d.G * d.TV * (d.TU + 1) * esz;
    return (b + 15) & ~(size_t)15;
}

// One tile of the transpose: tile index t (u fastest, then v, then slices);
// smem holds the tile.  NT: streaming stores.
template <typename C, int VU, int VV, bool NT = true>
__device__ __forceinline__ void xpose_tile(const C *__restrict__ in, C *__restrict__ out, const XposeDesc &d,
                                           uint32_t tile_index, unsigned char *smem)
{
    C *tile = reinterpret_cast<C *>(smem);

    const int TU = d.TU, TV = d.TV;
    const int ldt = TU + 1;
    uint32_t t = tile_index;
    const uint32_t tu = t % (uint32_t)d.tiles_u;
    t /= (uint32_t)d.tiles_u;
    const uint32_t tv = t % (uint32_t)d.tiles_v;
    const uint32_t tg = t / (uint32_t)d.tiles_v;
    const int64_t u0 = (int64_t)tu * TU, v0 = (int64_t)tv * TV, g0 = (int64_t)tg * d.G;
    const int nu = (int)min<int64_t>(TU, d.Nu - u0);
    const int nv = (int)min<int64_t>(TV, d.Nv - v0);
    const int ng = (int)min<int64_t>(d.G, d.nslices - g0);

    if (d.count) {
        // each wave publishes its sum at once: work left for the end of the
        // tile would delay the group's exit
        int moved = tile_moved(d, g0, ng, u0, nu, v0, nv);
        for (int off = 32; off > 0; off >>= 1) moved += __shfl_xor(moved, off);
        if ((threadIdx.x & 63) == 0 && moved)
            atomicAdd(d.counter + (tile_index % kCountSlots) * kCountStride, (unsigned long long)moved);
    }

    // load: rows (g, v) of contiguous u-values.  A thread's rows are taken
    // kTileBatch at a time, every load of a batch issued before any value
    // goes to LDS (a loop that writes each value as it arrives runs the
    // thread's loads one HBM round trip at a time).
    {
        const int per_row = TU / VU;
        const int tx = threadIdx.x % per_row;
        const int ty = threadIdx.x / per_row;
        const int ystep = kThreads / per_row;
        const int nrow = ng * nv;
        const int iu = tx * VU;
        const int spare = d.G * TV * ldt;  // first element after the tile
        int gcur = -1;
        int64_t abase = 0;
        for (int rb = ty; rb < nrow; rb += kTileBatch * ystep) {
            C val[kTileBatch][VU];
            int at[kTileBatch];
            // every item loads and writes, so that no load is left pending
            // from one trip to the next: an item past the tile loads an
            // element of the tile again (clamped) and writes it to the spare
            // 16 bytes after the tile, which the launchers reserve
#pragma unroll
            for (int j = 0; j < kTileBatch; ++j) {
                const int r = rb + j * ystep;
                const bool ok = r < nrow && iu < nu;
                const int rc = r < nrow ? r : nrow - 1;
                const int iuc = iu < nu ? iu : 0;
                const int g = rc / nv;
                const int iv = rc - g * nv;
                if (g != gcur) {
                    int c[3];
                    int64_t bb;
                    slice_coords(d, g0 + g, c, &abase, &bb);
                    gcur = g;
                }
                const C *p = in + abase + (v0 + iv) * d.a_sv + u0 + iuc;
                at[j] = ok ? (g * TV + iv) * ldt + iu : spare;
                if constexpr (VU == 2) {
                    const xf4 w = gld_nt(reinterpret_cast<const xf4 *>(p));
                    val[j][0] = mk<C>(w.x, w.y);
                    val[j][1] = mk<C>(w.z, w.w);
                } else {
                    val[j][0] = xld(p);
                }
            }
#pragma unroll
            for (int j = 0; j < kTileBatch; ++j) {
#pragma unroll
                for (int w = 0; w < VU; ++w) tile[at[j] + w] = val[j][w];
            }
        }
    }
    __syncthreads();

    // store: rows (g, u) of contiguous v-values, kTileBatch rows at a time,
    // every LDS read of a batch issued before its first store
    {
        const int per_row = TV / VV;
        const int tx = threadIdx.x % per_row;
        const int ty = threadIdx.x / per_row;
        const int ystep = kThreads / per_row;
        const int nrow = ng * nu;
        const int iv = tx * VV;
        int gcur = -1;
        int64_t bbase = 0;
        for (int rb = ty; rb < nrow; rb += kTileBatch * ystep) {
            C val[kTileBatch][VV];
            C *dst[kTileBatch];
#pragma unroll
            for (int j = 0; j < kTileBatch; ++j) {
                const int r = rb + j * ystep;
                dst[j] = nullptr;
                if (r < nrow && iv < nv) {
                    const int g = r / nu;
                    const int iu = r - g * nu;
                    if (g != gcur) {
                        int c[3];
                        int64_t ab;
                        slice_coords(d, g0 + g, c, &ab, &bbase);
                        gcur = g;
                    }
                    dst[j] = out + bbase + (u0 + iu) * d.b_su + v0 + iv;
                    const C *tcol = tile + (g * TV + iv) * ldt + iu;
                    val[j][0] = tcol[0];
                    if constexpr (VV == 2) val[j][1] = tcol[ldt];
                }
            }
#pragma unroll
            for (int j = 0; j < kTileBatch; ++j)
                if (dst[j]) {
                    if constexpr (VV == 2) {
                        const xf4 w = {val[j][0].x, val[j][0].y, val[j][1].x, val[j][1].y};
                        if constexpr (NT)
                            gst_nt(w, reinterpret_cast<xf4 *>(dst[j]));
                        else
                            gst(w, reinterpret_cast<xf4 *>(dst[j]));
                    } else {
                        xst<NT>(dst[j], val[j][0]);
                    }
                }
        }
    }
    __syncthreads();  // the LDS block may be reused by the caller's next unit
}

}  // namespace fftrw
