// fft_ct_launch.hip -- table of the compile-time row FFT kernels (fft_ct.hip),
// the launch shapes of the fused kernel, and the launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "fft_ct.hpp"
#include "fft_ct_table.hpp"

namespace fftrw {

int ct_part_0(CtEntry *);
int ct_part_1(CtEntry *);
int ct_part_2(CtEntry *);
int ct_part_3(CtEntry *);
int ct_part_4(CtEntry *);
int ct_part_5(CtEntry *);
int ct_part_6(CtEntry *);
int ct_part_7(CtEntry *);
int ct_part_8(CtEntry *);
int ct_part_9(CtEntry *);
int ct_part_10(CtEntry *);
int ct_part_11(CtEntry *);
int ct_part_12(CtEntry *);
int ct_part_13(CtEntry *);
int ct_part_14(CtEntry *);
int ct_part_15(CtEntry *);

namespace {

struct CtTable {
    CtEntry e[2 * kCtLengths];
    const CtEntry *by_n[2][kCtMax + 1] = {};
    CtTable()
    {
        int n = 0;
        for (auto part : {ct_part_0, ct_part_1, ct_part_2, ct_part_3, ct_part_4, ct_part_5, ct_part_6, ct_part_7,
                          ct_part_8, ct_part_9, ct_part_10, ct_part_11, ct_part_12, ct_part_13, ct_part_14,
                          ct_part_15})
            n += part(e + n);
        for (int i = 0; i < n; ++i) by_n[e[i].esz == 16][e[i].N] = &e[i];
    }
};

const CtEntry *find(int N, bool fp64)
{
    static const CtTable table;
    return N >= 2 && N <= kCtMax ? table.by_n[fp64][N] : nullptr;
}

constexpr size_t kLdsBytes = 160 * 1024;  // of one compute unit

// whether the array (half of the L2s' 32 MB and a little more) mostly stays in
// the L2s between steps
bool ct_small(const XposeDesc &d, int esz) { return d.Nu * d.Nv * d.nslices * esz <= ((int64_t)20 << 20); }

// n / d for n < 2^31 (see CtDiv)
CtDiv make_div(int64_t d)
{
    if (d <= 1) return {0, 0, ~0u};
    uint32_t l = 0;
    while (((int64_t)1 << l) < d) ++l;
    return {(uint32_t)(((uint64_t)1 << (31 + l)) / (uint64_t)d + 1), l - 1, 0};
}

// Shape of a fused step: the
// work-group size with the best score, the product of
//   * the share of its row places that rows fill;
//   * 0.8, 0.5 or 0.25 for runs under 128, 64 or 32 bytes, and 0.93 for runs
//     under 256 bytes where runs start inside a 128-byte line: 512^3 with
//     64-byte runs took 1598 against 1193 us per transform with 128-byte ones,
//     60x48x50x45 took 95 us in 128-byte and 88 us in whole-axis runs;
//   * (units / 256)^1/2 for fewer units than compute units;
//   * 0.9 when only one group fits a compute unit.
// Ties go to the smaller group: one wave needs no barrier (64^4: 186 us in
// groups of one wave, 192 us in groups of four).
bool ct_shape(const CtEntry &e, const XposeDesc &d, CtStep *best)
{
    const int64_t nv = d.Nv, ns = d.nslices;
    double top = -1;
    const int line = 128 / e.esz;
    const bool lines = d.Nv % line == 0;  // runs of whole lines start on one
    for (int threads = e.min_threads; threads <= e.max_threads; threads *= 2) {
        const int rows = threads / e.L;
        CtStep c;
        c.e = &e;
        c.threads = threads;
        while ((1 << c.s.lr) < rows) ++c.s.lr;
        if (nv <= rows) {
            c.s.rw = (int)nv;
            c.s.G = (int)std::min<int64_t>(rows / nv, ns);
        } else {
            c.s.G = 1;
            c.s.rw = rows;
            for (int r = line; r < rows; r += line)
                if ((nv + r - 1) / r <= (nv + rows - 1) / rows) {
                    c.s.rw = r;
                    break;
                }
        }
        // LDS: the rows' exchange buffers and the output block share it, then
        // the tables of slice and row bases.  The block's lines get one value
        // of padding per 128 bytes, or none beyond what positions need where
        // it would not fit.
        const size_t tables = (size_t)c.s.G * 8 + (e.staged ? (size_t)rows * 8 : 0);
        auto data = [&](int sp) {
            return ((size_t)std::max(rows * e.pitch, e.N * sp) * e.esz + 15) & ~(size_t)15;
        };
        c.s.sp = rows + std::max(1, rows / line);
        if (data(c.s.sp) + tables > kLdsBytes) c.s.sp = rows + (rows - 1) / line;
        c.s.tab = (uint32_t)data(c.s.sp);
        c.lds = c.s.tab + tables;
        if (c.lds > kLdsBytes) break;
        c.s.tiles_v = (uint32_t)((nv + c.s.rw - 1) / c.s.rw);
        c.units = (int64_t)c.s.tiles_v * ((ns + c.s.G - 1) / c.s.G);
        double score = (double)nv * ns / ((double)c.units * rows);
        const int run = c.s.rw * e.esz;
        if (c.s.rw < nv) score *= run < 32 ? 0.25 : run < 64 ? 0.5 : run < 128 ? 0.8 : run < 256 && !lines ? 0.93 : 1;
        if (c.units < 256) score *= std::sqrt((double)c.units / 256);
        if (c.lds * 2 > kLdsBytes) score *= 0.9;
        if (score > top) {
            top = score;
            *best = c;
        }
    }
    if (top < 0 || best->units >= (int64_t)0x7ffffff0) return false;
    CtShape &s = best->s;
    s.units = (uint32_t)best->units;
    s.dtv = make_div(s.tiles_v);
    for (int i = 0; i < 3; ++i) s.db[i] = make_div(i < d.nbat ? d.bsize[i] : 1);
    // Every run made of whole 128-byte lines?
    best->whole = lines && (s.rw % line == 0 || s.rw == d.Nv);
    // Neighbouring units on one XCD, whose L2 then joins the parts of a line:
    // where runs are not made of whole 64-byte sectors (4096x2048 with 32-byte
    // runs: 83 against 110 us; 64-byte runs lose a little: 1024x1024 17.9
    // against 18.9 us), and for arrays that the L2s hold (128^3: 24.7 against
    // 27.4 us; 64^4 loses 5%).
    const int sector = 64 / e.esz;
    const bool sectors = d.Nv % sector == 0 && (s.rw % sector == 0 || s.rw == d.Nv);
    best->grid = s.units;
    if ((!sectors || (best->whole && ct_small(d, e.esz))) && s.units > 64) {
        s.per_xcd = (s.units + 7) / 8;
        best->grid = s.per_xcd * 8;
    }
    return true;
}

}  // namespace

bool ct_supported(int N, bool fp64) { return find(N, fp64) != nullptr; }

// Describe the kernel for N: number of twiddle entries and the radix list.
void ct_describe(int N, bool fp64, int *tw_count, int *radices, int *npass)
{
    const CtEntry &e = *find(N, fp64);
    *tw_count = e.tw_count;
    *npass = e.np;
    for (int i = 0; i < e.np; ++i) radices[i] = e.r[i];
}

struct CtRadices {
    int r[5];
    int n;
};

// per-pass twiddle table, FP64 arithmetic: pass p holds w_{Ns R}^{i k} at
// [i - 1][k], i = 1..R-1, k < Ns (nothing for the first pass: k = 0)
template <typename C> __global__ void __launch_bounds__(kThreads) ct_twiddle_kernel(C *out, CtRadices ra)
{
    const int idx = blockIdx.x * kThreads + threadIdx.x;
    int off = 0, Ns = ra.r[0];
    for (int p = 1; p < ra.n; ++p) {
        const int R = ra.r[p], cnt = Ns * (R - 1);
        if (idx >= off && idx < off + cnt) {
            const int i = (idx - off) / Ns + 1, k = (idx - off) % Ns;
            const int n = Ns * R;
            double s, c;
            unit_root((i * k) % n, n, &c, &s);
            out[idx] = mk<C>((typename RealOf<C>::type)c, (typename RealOf<C>::type)s);
        }
        off += cnt;
        Ns *= R;
    }
}

hipError_t ct_make_twiddles(int N, bool fp64, void *tw, hipStream_t s)
{
    const CtEntry &e = *find(N, fp64);
    if (e.tw_count == 0) return hipSuccess;
    CtRadices ra{};
    ra.n = e.np;
    for (int i = 0; i < e.np; ++i) ra.r[i] = e.r[i];
    const dim3 grid((unsigned)((e.tw_count + kThreads - 1) / kThreads));
    if (fp64)
        hipLaunchKernelGGL(ct_twiddle_kernel<double2>, grid, dim3(kThreads), 0, s, (double2 *)tw, ra);
    else
        hipLaunchKernelGGL(ct_twiddle_kernel<float2>, grid, dim3(kThreads), 0, s, (float2 *)tw, ra);
    return hipGetLastError();
}

// The form (XposeDesc::count) in which groups of `threads` beside a step's own
// count its transpose, 0 if that needs a launch apart.  Split rows (A's owner
// changes along u or B's along v) are counted beside the step while every
// thread of the groups has one piece at most, which the step hides (128^3 at
// 16,385 processes 26 us, 64 apart); more pieces fill the chip by themselves
// (256^3, one process per point: 856 us apart, 23 ms on groups for whole rows).
int count_beside(const XposeDesc &d, int threads)
{
    bool split = false;
    for (int j = 0; j < d.ka; ++j) split = split || d.srca[j] == 4;
    for (int j = 0; j < d.kb; ++j) split = split || d.srcb[j] == 3;
    if (!split) return 1;
    const int64_t rows = d.nslices * d.Nv, pieces = count_pieces(d);
    if (rows > (int64_t)kCountBlock * threads / pieces) return 0;
    int lg = 0;
    while ((2 << lg) < pieces) ++lg;
    return 2 + lg;
}

// a transpose's owner changes alone: one word of the counter per group, so
// large groups where rows are split
constexpr int kCountThreads = 1024;
__global__ void __launch_bounds__(kCountThreads) count_kernel(const XposeDesc d)
{
    __shared__ unsigned long long part[kCountThreads / 64];
    count_share(d, blockIdx.x, gridDim.x, part);
}

hipError_t launch_count(const XposeDesc &d, hipStream_t s)
{
    XposeDesc x = d;
    int threads = kThreads;
    x.count = count_beside(d, threads);
    if (!x.count) {
        // two items for every thread the chip holds, or a piece per item
        threads = kCountThreads;
        const int64_t items = 2 * (int64_t)kCountBlock * threads, pieces = count_pieces(d);
        int lg = 0;
        while (((d.nslices * d.Nv) << lg) < items && (2 << lg) < pieces) ++lg;
        x.count = 2 + lg;
    }
    hipLaunchKernelGGL(count_kernel, dim3(count_groups(x, threads)), dim3(threads), 0, s, x);
    return hipGetLastError();
}

// the launch of a fused step, false if the kernel has no shape for it
bool ct_plan_step(int N, bool fp64, const XposeDesc &d, CtStep *step)
{
    const CtEntry *e = find(N, fp64);
    return e && ct_shape(*e, d, step);
}

hipError_t launch_ct_fused(const CtStep &step, const void *tw, const XposeDesc &d, int dir, const void *in, void *out,
                           double scale, CachePolicy policy, hipStream_t s)
{
    if (step.units <= 0) return hipSuccess;
    CtShape c = step.s;
    c.nt_load = policy.nt_load;
    c.nt_store = policy.nt_store;
    c.inverse = dir > 0;
    c.do_scale = scale != 1.0;
    const int ncount = d.count ? count_groups(d, step.threads) : 0;
    hipLaunchKernelGGL(step.e->fused, dim3(step.grid + ncount), dim3(step.threads), step.lds, s, in, out, d, c, tw, scale,
                       ncount);
    return hipGetLastError();
}

// Rows alone that pass through LDS in the fused kernels go straight between
// HBM and registers in a small array, where the way through LDS is latency
// (64 points, 4 MB 0.81 of the time; 32 MB 0.73 to 1.9 times, by the length);
// rows of several whole lines up to 12 MB (through LDS / straight: 64 points,
// 12 MB 6.3 / 4.6 us, complex128 40 points, 12 MB 7.3 / 5.5; but 48 points,
// 16 MB 7.4 / 11.0, and rows of 256 bytes, 12 MB 1.0 to 1.9 times).
constexpr int64_t kStraightBytes = 4 << 20, kStraightLineBytes = 12 << 20;

// Rows that are not whole lines are copied as one block per group where the
// array is too large for the Infinity Cache to join the lines' parts (729^3,
// 3.1 GB: 1583 us row by row, 1226 as blocks), and where rows are short and odd
// (125 points, 131 MB: 47 and 43 us; longer rows and pairs of values lose:
// 625 points 39 and 42).
constexpr int64_t kBlockRowBytes = 1024, kBlockBytes = (int64_t)256 << 20;

constexpr int64_t kFewGroups = 448;

hipError_t launch_ct_rows(int N, bool fp64, const void *tw, int64_t nrows, int dir, const void *in, void *out,
                          double scale, CachePolicy policy, hipStream_t s)
{
    const CtEntry *e = find(N, fp64);
    if (!e) return hipErrorInvalidValue;
    if (nrows <= 0) return hipSuccess;
    CtRowsShape c{};
    // groups of 256 threads, or smaller ones where the chip then holds more
    // waves (625 points, whose padded rows leave LDS for two groups of 256
    // threads: 42.7 us for 134 MB, 39.2 in groups of 64) or would have few groups
    // (128 points, 256 threads / fewer: 1 MB 3.72 / 3.12 us, 12 MB, 1.4 groups a
    // compute unit, 6.72 / 5.56, but 16 MB, 1.9 groups, 6.32 / 7.24).  Rows of one
    // lane that all fit one group stay in it (256 rows of 4 points 1.48 / 1.76).
    auto resident = [&](int t) {
        return std::min<int64_t>((int64_t)(kLdsBytes / ((size_t)(t / e->L) * e->pitch * e->esz)) * t, 1024);
    };
    int threads = std::max(256, e->min_threads);
    while (threads > e->min_threads &&
           (resident(threads / 2) > resident(threads) ||
            (nrows * e->L / threads < kFewGroups && (e->L > 1 || nrows > threads))))
        threads /= 2;
    const int rows = threads / e->L;
    while ((1 << c.lr) < rows) ++c.lr;
    const int64_t grid = (nrows + rows - 1) / rows;
    if (grid >= (int64_t)0x7fffffff) return hipErrorInvalidValue;
    const int64_t row = (int64_t)N * e->esz, bytes = nrows * row;
    const bool block = e->rows_block && (bytes > kBlockBytes || (N % 2 != 0 && row < kBlockRowBytes));
    const bool lines = row % 128 == 0 && row > 256;
    const bool straight = e->rows_straight && bytes <= (lines ? kStraightLineBytes : kStraightBytes);
    // (parts of lines are left to the caches to join)
    const bool nt_store = policy.nt_store && (block || straight || row % 128 == 0 || 128 % row == 0);
    c.flags = (policy.nt_load ? kCtNtLoad : 0) | (nt_store ? kCtNtStore : 0) | (dir > 0 ? kCtInverse : 0) |
              (scale != 1.0 ? kCtScale : 0);
    hipLaunchKernelGGL(straight ? e->rows_straight : block ? e->rows_block : e->rows, dim3((unsigned)grid), dim3(threads),
                       (size_t)rows * e->pitch * e->esz, s, in, out, nrows, tw, scale, c);
    return hipGetLastError();
}

}  // namespace fftrw
