// fft_ct_table.hpp -- the row lengths with compile-time kernels and the record
// the host keeps of each.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace fftrw {

// Every 2,3,5-smooth length from 2 to kCtMax (complex64) or kCtMaxFp64
// (complex128).  Plans accept lengths up to 4096 in both: complex128 rows past
// kCtMaxFp64 run the run-time-radix kernel, in plans of separate kernels.
constexpr int kCtMax = 4096;
constexpr int kCtMaxFp64 = 2048;

constexpr bool ct_smooth(int n)
{
    while (n % 2 == 0) n /= 2;
    while (n % 3 == 0) n /= 3;
    while (n % 5 == 0) n /= 5;
    return n == 1;
}

struct CtLengthTable {
    int count = 0;
    int n[256] = {};
};

constexpr CtLengthTable ct_make_lengths()
{
    CtLengthTable t;
    for (int n = 2; n <= kCtMax; ++n)
        if (ct_smooth(n)) t.n[t.count++] = n;
    return t;
}

constexpr CtLengthTable kCtLengthTable = ct_make_lengths();
constexpr int kCtLengths = kCtLengthTable.count;
constexpr int ct_length(int i) { return kCtLengthTable.n[i]; }

// Exact n / d for n < 2^31 by a multiply: m = floor(2^(31 + l) / d) + 1 with
// l = ceil(log2 d) exceeds 2^(31 + l) / d by at most 1, which adds at most
// n / 2^(31 + l) < 1 / 2^l <= 1 / d to n / d.  (d = 1: m = 0, one = ~0.)
struct CtDiv {
    uint32_t m, s, one;
    __device__ __forceinline__ uint32_t operator()(uint32_t n) const { return (__umulhi(n, m) + (n & one)) >> s; }
};

// run-time shape of a launch
struct CtShape {
    int lr;                 // log2 of the rows per work-group
    int rw, G;              // rows consecutive in v per slice, slices per work-group
    uint32_t tiles_v;       // v-blocks per group of slices
    uint32_t units;         // work-groups with work
    uint32_t per_xcd;       // > 0: consecutive units run on one XCD, this many each
    uint32_t tab;           // byte offset of the base tables in LDS
    int sp;                 // LDS pitch of the output block's frequencies
    int nt_load, nt_store;  // streaming (non-temporal) HBM accesses
    int inverse;            // conjugate in and out: the inverse by the forward's passes
    int do_scale;
    CtDiv dtv, db[3];       // divisions by tiles_v and by the batch axes' sizes
};

// ... of rows alone (few bytes: a small transform waits for its arguments)
struct CtRowsShape {
    int lr;             // as above
    uint32_t flags;     // kCtNtLoad ..
};
constexpr uint32_t kCtNtLoad = 1, kCtNtStore = 2, kCtInverse = 4, kCtScale = 8;

using CtFusedKernel = void (*)(const void *, void *, const XposeDesc, const CtShape, const void *, double, int);
using CtRowsKernel = void (*)(const void *, void *, int64_t, const void *, double, const CtRowsShape);

struct CtEntry {
    int N, esz;
    int L, np, r[5];
    int tw_count;
    int min_threads, max_threads;  // powers of two
    int pitch;   // LDS pitch of a row (values)
    int staged;  // rows go through LDS first (and need a table of row bases)
    CtFusedKernel fused;
    CtRowsKernel rows;
    CtRowsKernel rows_block;     // rows that are not whole lines, as one block (else null)
    CtRowsKernel rows_straight;  // rows otherwise staged in LDS, without (else null)
};

// a fused step's launch, made once per plan
struct CtStep {
    const CtEntry *e = nullptr;
    CtShape s{};
    int threads = 0;
    unsigned grid = 0;
    size_t lds = 0;
    int64_t units = 0;
    bool whole = false;  // every run is made of whole 128-byte lines
};

}  // namespace fftrw
