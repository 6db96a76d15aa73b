// batch.hip -- many uneven transforms in one persistent launch.
//
// Each item is a whole Fig. 4 pipeline (M FFT steps and M transposes) with its
// own sizes, process count and order.  The work of all items is cut into
// units -- a block of rows of one FFT step, or a tile of one transpose --
// grouped into stage levels: level s holds stage s of every item that has
// one.  One grid of work-groups, sized to stay resident, sweeps the levels:
// units are taken from one atomic counter, a few consecutive units per claim,
// level after level.  A work-group leaves a level once its next claim is of a
// later one; the last group to leave on an XCD writes that XCD's L2 back
// (a release at device scope) and adds the units its groups completed to the
// level's done counter, and whoever completes that counter opens the next
// level, for which the groups wait on copies of one word (then acquire, so
// data written on one XCD is seen on the others).  This keeps every item's
// FFT -> transpose -> FFT order.  Counting units rather than arrivals means
// no work-group waits for one that has not started: a unit is only ever
// claimed by a running work-group, and a level is left only once all its
// units are claimed, so the wait ends whether or not the whole grid is
// resident (another kernel may hold part of the device).  Waiting polls a
// device-coherent word without invalidating caches, and every wait is
// bounded by the real-time clock: past the bound the work-group adds one to
// a sticky time-out count and goes on, so the grid always drains and the
// host can refuse the result.
//
// What the levels cost: same-address atomics take 11.5 ns each, and 1024
// groups that each release or acquire at device scope 7.5 us, so a level's
// end can cost a small batch more than its units.  With one release per XCD
// instead of per group, no claim made in vain, no more groups than units and
// the waiters off the counters' lines, one 96^3 transform takes 64 us instead
// of 224, sixteen 64^3 153 instead of 378, 32 items of 9 x 10^3 to 4 x 10^6
// points 572 instead of 854 and 256 of them 3.44 ms instead of 3.69
// (complex64).  Eight claim counters, one per XCD, take the small ones
// further (53 and 125 us) and the large ones back (590 us, 3.59 ms): the
// search for units left elsewhere costs every unit registers and
// instructions.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

#include "../../include/fftrw.h"
#include "decomp.hpp"
#include "errors.hpp"
#include "fft_generic.hpp"
#include "fused_generic.hpp"
#include "kernels.hpp"
#include "plan.hpp"
#include "tune.hpp"
#include "xpose_tile.hpp"

namespace fftrw {

constexpr int kMaxStages = 2 * kMaxDims;

struct BatchItemDev {
    float2 *buf[3];                 // 0 in (read only), 1 out, 2 work
    int M;
    int nstage;                     // 2M (2M - 1 with LEAVE_PERMUTED); fused: M
    int fused;                      // stage t = FFT step t fused with transpose t
    int nx;                         // transposes executed (M, or M - 1 with LEAVE_PERMUTED)
    int frw[kMaxDims];              // rows (consecutive v) per slice of a fused unit of stage t
    int fg[kMaxDims];               // slices per fused unit of stage t
    int src[kMaxStages];            // 0 in, 1 out, 2 work
    int dst[kMaxStages];
    int64_t prefix[kMaxStages + 1]; // units of this item before stage s
    float inv_scale;                // 1/T for the inverse's last FFT step
    int xv[kMaxDims];               // 16-byte access flags of transpose t: bit0 u, bit1 v
    FftDesc fft[kMaxDims];
    XposeDesc xp[kMaxDims];
};

struct BatchTask {
    int item, stage;
    int64_t unit0, nunits;  // unit0 counts from the start of the task's level
};

// A claim takes 2^kClaimLog units, and single units for a level's last
// kClaimTail per work-group.
constexpr int kClaimLog = 2;
constexpr int kClaimTail = 4;

// zeroed before every launch, one per level: the claim counter (level 0's
// serves every level), a counter of completed units, copies of the word that
// opens the next level, and a word per XCD (bits 63:48 groups that entered
// the level, 47:32 groups that left it, 31:0 their completed units not yet in
// `done`), each on a 128-byte line of its own
constexpr int kCtrLine = 16;     // 64-bit words per line
constexpr int kOpenCopies = 32;
constexpr int kMaxXcds = 16;
struct BatchLevelCtr {
    unsigned long long next[kCtrLine];
    unsigned long long done[kCtrLine];
    unsigned long long open[kOpenCopies][kCtrLine];
    unsigned long long xcd[kMaxXcds][kCtrLine];
};
constexpr unsigned long long kEntered = 1ull << 48, kLeft = 1ull << 32;

// the XCD this wave runs on: bits 3:0 of hardware register 20 (XCC_ID)
__device__ __forceinline__ int xcd_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)); }

// task starts of one level held in LDS for the per-unit search
constexpr int kLevelTasksLds = 256;

// s_waitcnt operand: vector memory count 0 (bits 3:0 and 15:14), the export
// and LDS/scalar counts at their maxima (bits 6:4 and 11:8)
constexpr int kWaitVmcnt0 = 0x0F70;

// real-time clock ticks (100 MHz) a work-group may wait at one barrier
constexpr unsigned long long kWaitTicks = 200000000ull;

// Takes the next unit index from a level's claim counter (a 64-bit word
// whose low half counts; levels hold fewer than 2^32 units).  A wrapping
// increment rather than an add: the compiler rewrites a single lane's atomic
// add into a wave-wide scan that needs the result at once, which would wait
// for every load and store the wave has in flight; the increment's result is
// waited for only where it is used.
__device__ __forceinline__ unsigned claim(unsigned long long *ctr)
{
    return __builtin_amdgcn_atomic_inc32(reinterpret_cast<unsigned *>(ctr), 0xffffffffu, __ATOMIC_RELAXED, "agent");
}

// The buffer of a stage.  One uniform address, read through the scalar
// cache: a vector load would count on the wait counter that the unit's HBM
// stores also count on, and waiting for it would wait for the previous
// unit's stores as well.
__device__ __forceinline__ float2 *batch_buf(const BatchItemDev &it, int kind)
{
    return it.buf[__builtin_amdgcn_readfirstlane(kind)];
}

// Without LEAN the kernel is held to three waves per SIMD (at most 168 VGPRs;
// the stage kernels need a few more otherwise, which would leave two: 256
// uneven items 3.23 -> 4.10 ms with LEAVE_PERMUTED, 5.70 -> 6.79 with
// BATCH_NO_FUSE, with radix 16 compiled in as well, which no step has).
// LEAN: every stage of every item is a fused unit with radices 2 to 6 and 8
// only, and every item's buffers hold fewer than 2^32 bytes (32-bit offsets);
// without the other stage kernels and the larger passes the kernel fits four
// waves per SIMD.
template <int DIR, bool TW_LDS, bool LEAN>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(LEAN ? 4 : 3)))
    batch_kernel(const BatchItemDev *__restrict__ items, const BatchTask *__restrict__ tasks,
                 const int *__restrict__ level_task0, const int64_t *__restrict__ level_units, int nlevels,
                 BatchLevelCtr *ctr, unsigned long long *timeouts, unsigned long long wait_ticks)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_unit0[kLevelTasksLds];
    __shared__ int s_unit, s_task, s_end;
    unsigned pending = 0;     // thread 0: its claim in flight
    unsigned claims0 = 0;     // claims of the levels before this one
    const int xcd = xcd_id();
    if (threadIdx.x == 0) {
        atomicAdd(&ctr[0].xcd[xcd][0], kEntered);
        pending = claim(&ctr[0].next[0]);
    }
    for (int lv = 0; lv < nlevels; ++lv) {
        const int64_t nunits = level_units[lv];
        const int t0 = level_task0[lv], t1 = level_task0[lv + 1];
        // the level's task starts, searched in LDS when they fit
        const bool in_lds = t1 - t0 <= kLevelTasksLds;
        if (in_lds)
            for (int i = threadIdx.x; i < t1 - t0; i += kThreads) s_unit0[i] = (int)tasks[t0 + i].unit0;
        __syncthreads();
        // Thread 0 claims units and finds each one's task (a binary search
        // over the level's task starts, skipped while the units stay in one
        // task).  A claim takes a chunk of consecutive units, and a single
        // unit for the level's last kClaimTail x grid, so that few atomics
        // reach the counter (they take 11.5 ns each whoever issues them) and
        // the level still ends evenly.  The levels' claims are numbered
        // through: a claim past a level's end is one of the next level, kept
        // over the barrier, so that no claim is made in vain and none is
        // waited for when a level starts.  A unit's successor is handed to
        // the work-group (s_unit, s_task) in the middle of the unit, once the
        // unit's own row loads have arrived, and a new chunk is claimed when
        // the last unit of the current one starts: loads, stores and atomics
        // count on one wait counter in issue order, so reading a claim at
        // the next unit's start would also wait for this unit's stores.
        // (a level has fewer than 2^31 units and the launch, with one claim
        // past its end per work-group, fewer than 2^32 claims)
        const int nu32 = (int)nunits;
        const int tail = min(nu32, (int)gridDim.x * kClaimTail);
        const unsigned nchunk = (unsigned)(nu32 - tail) >> kClaimLog;
        const unsigned head = nchunk << kClaimLog;
        // Thread 0 keeps the unit being run and its task in s_unit and s_task
        // (which the work-group reads), the end of its chunk in s_end, and
        // the claim in flight in a register.
        unsigned ndone = 0;
        // thread 0: publish unit `cur` of chunk end `end`, its task searched
        // from task index `task` (counted from t0) on
        auto publish_unit = [&](int cur, int end, int task) {
            const int last = t1 - t0 - 1;
            if (cur < nu32 && task < last &&
                cur >= (in_lds ? s_unit0[task + 1] : (int)tasks[t0 + task + 1].unit0)) {
                int lo = task + 1, hi = last;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if ((in_lds ? s_unit0[mid] : (int)tasks[t0 + mid].unit0) <= cur)
                        lo = mid;
                    else
                        hi = mid - 1;
                }
                task = lo;
            }
            s_unit = cur;
            s_end = end;
            s_task = t0 + task;
        };
        // thread 0: the first unit of the claim in flight, or unit nunits
        auto publish_chunk = [&](int task) {
            const unsigned c = pending - claims0;
            const bool whole = c < nchunk;
            const unsigned cur = whole ? c << kClaimLog : min(head + (c - nchunk), (unsigned)nu32);
            publish_unit((int)cur, (int)(cur + (whole ? 1u << kClaimLog : 1u)), task);
        };
        auto publish = [&]() {
            if (threadIdx.x == 0) {
                const int cur = s_unit, end = s_end, task = s_task - t0;
                if (cur + 1 < end)
                    publish_unit(cur + 1, end, task);
                else
                    publish_chunk(task);
            }
        };
        if (threadIdx.x == 0) publish_chunk(0);
        __syncthreads();
        for (;;) {
            // every unit function synchronises the work-group before it calls
            // publish (and non-fused units are preceded by a barrier), so these
            // reads are done before thread 0 overwrites the values
            const int u = s_unit, lo = s_task;
            if (u >= nu32) break;
            if (threadIdx.x == 0) {
                ++ndone;
                if (u + 1 >= s_end) pending = claim(&ctr[0].next[0]);
            }
            const BatchTask tk = tasks[lo];
            const BatchItemDev &it = items[tk.item];
            const int64_t local = u - tk.unit0;
            const int st = tk.stage;
            const float2 *src = batch_buf(it, it.src[st]);
            float2 *dst = batch_buf(it, it.dst[st]);
            if constexpr (LEAN) {
                const bool last = st == it.M - 1;
                fft_xpose_unit<float2, DIR, TW_LDS, kRadBatch, true, true>(src, dst, it.fft[st], it.xp[st], it.frw[st], it.fg[st],
                                                                local,
                                                                DIR > 0 && last ? it.inv_scale : 1.f, DIR > 0 && last,
                                                                smem, publish);
                continue;
            }
            if (it.fused && st < it.nx) {
                const bool last = st == it.M - 1;
                fft_xpose_unit<float2, DIR, TW_LDS, kRadBatch, false, true>(
                    src, dst, it.fft[st], it.xp[st], it.frw[st], it.fg[st], local,
                    DIR > 0 && last ? it.inv_scale : 1.f, DIR > 0 && last, smem, publish);
                continue;
            }
            // the other unit kinds take the next unit before they start
            __syncthreads();
            publish();
            if (it.fused) {
                const bool last = st == it.M - 1;
                fft_rows_block<float2, DIR, kRadBatch>(src, dst, it.fft[st], local, DIR > 0 && last ? it.inv_scale : 1.f,
                                            DIR > 0 && last, reinterpret_cast<float2 *>(smem));
                continue;
            }
            const int t = st >> 1;
            if ((st & 1) == 0) {
                const bool last = t == it.M - 1;
                fft_rows_block<float2, DIR, kRadBatch>(src, dst, it.fft[t], local, DIR > 0 && last ? it.inv_scale : 1.f,
                                            DIR > 0 && last, reinterpret_cast<float2 *>(smem));
            } else {
                switch (it.xv[t]) {
                case 3: xpose_tile<float2, 2, 2>(src, dst, it.xp[t], (uint32_t)local, smem); break;
                case 1: xpose_tile<float2, 2, 1>(src, dst, it.xp[t], (uint32_t)local, smem); break;
                case 2: xpose_tile<float2, 1, 2>(src, dst, it.xp[t], (uint32_t)local, smem); break;
                default: xpose_tile<float2, 1, 1>(src, dst, it.xp[t], (uint32_t)local, smem); break;
                }
            }
        }
        if (lv + 1 == nlevels) break;
        claims0 += nchunk + ((unsigned)nu32 - head);
        // Level barrier: publish the units this group completed, wait for
        // all.  Every wave first waits until its own stores have completed
        // (they are then in the L2; a workgroup-scope release does not wait
        // for them); the agent-scope fences are issued by thread 0's wave
        // alone: a release writes back the L2 (whatever wave of the XCD wrote
        // the lines) before the count is published, and the acquire
        // invalidates the L2 and this CU's L1, which the group's other waves
        // read through after the second barrier.  The group that finds the
        // XCD's entered and left counts equal takes the units counted there;
        // a group that enters later finds them equal again when it leaves and
        // takes its own.
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (threadIdx.x == 0) {
            atomicAdd(&ctr[lv + 1].xcd[xcd][0], kEntered);
            unsigned long long *mine = &ctr[lv].xcd[xcd][0];
            const unsigned long long now = atomicAdd(mine, kLeft + ndone) + kLeft + ndone;
            bool open = nunits == 0;
            if ((now >> 48) == ((now >> 32) & 0xffff)) {
                const unsigned long long n = atomicAnd(mine, ~0xffffffffull) & 0xffffffffull;
                if (n) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    if (atomicAdd(&ctr[lv].done[0], n) + n == (unsigned long long)nunits) {
                        // the level's last units: every XCD's stores are in
                        // memory before its count, the counts before this
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
                        for (int i = 0; i < kOpenCopies; ++i)
                            __hip_atomic_store(&ctr[lv].open[i][0], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        open = true;
                    }
                }
            }
            const unsigned long long *word = &ctr[lv].open[blockIdx.x % kOpenCopies][0];
            const unsigned long long w0 = wall_clock64();
            while (!open && !__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                if (wall_clock64() - w0 > wait_ticks) {
                    atomicAdd(timeouts, 1ull);
                    break;
                }
                __builtin_amdgcn_s_sleep(4);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
    }
}

__global__ void batch_reset_kernel(unsigned long long *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

}  // namespace fftrw

// ---- host side ----------------------------------------------------------------
namespace fftrw {

int plan_create(fft_plan_t *plan, int M, const int64_t *dims, int64_t P, const int8_t *order, int dtype,
                int precision, unsigned flags, bool generic_rows, const TuneTable *tune, DevArena *arena);
void plan_free(fft_plan_t plan);
int factor_radices(int64_t n, int *rad);

struct fft_batch_impl {
    int n = 0;
    unsigned flags = 0;
    std::vector<fft_plan_t> plans;
    std::vector<BatchItemDev> h_items;
    std::vector<BatchTask> h_tasks;
    BatchItemDev *d_items = nullptr;
    BatchTask *d_tasks = nullptr;
    unsigned long long *d_ctr = nullptr;  // a BatchLevelCtr per level, then moved[sum of M_i]
    unsigned long long *d_timeouts = nullptr;  // sticky count of timed-out waits (never reset)
    bool timed_out = false;               // a stats call has seen d_timeouts != 0
    unsigned long long wait_ticks = kWaitTicks;  // bound of one level wait (real-time clock ticks)
    int64_t nctr = 0;
    std::vector<int> level_task0;         // first task of each level (+ end)
    std::vector<int64_t> level_units;     // units of each level
    int *d_level_task0 = nullptr;
    int64_t *d_level_units = nullptr;
    std::vector<int64_t> moved_off;       // first moved counter of each item
    int64_t total = 0;
    int grid = 0;
    size_t lds = 0;
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph[2] = {nullptr, nullptr};
    hipGraphExec_t gexec[2] = {nullptr, nullptr};
    bool pointers_set = false;
    bool tuned = false;  // a matching autotuner cache was applied
    bool any_fused = false;
    bool tw_lds = false;  // fused units stage their twiddle tables in LDS
    bool lean = false;    // every stage a fused unit of radices 2 to 6 and 8 (batch_kernel's LEAN form)
};

// Radices of a batch's step of built-in order: of 2..6 and 8 the fewest
// passes, then the smallest sum, those with fewer factors 2 first (a first
// pass of radix r stores with a stride of r values, and strides of many
// factors 2 meet on the LDS banks).  A lane holds 16 to 20 values whatever
// the radix, so 6 and 8 cost the LEAN kernel no wave: 256 uneven items 2.97
// -> 2.90 ms, 4 x 256^3 1.06 -> 0.92, sixteen 64^3 152 -> 134 us (64 x 60^3
// 237 -> 240).  With 9 and 10 as well it spills and takes 3.09 ms.
int batch_radices(i64 n, int *rad)
{
    int best[kMaxPasses], nbest = kMaxPasses + 1, sbest = 0, cur[kMaxPasses];
    std::function<void(i64, int, int, int)> go = [&](i64 left, int np, int sum, int top) {
        if (left == 1) {
            if (np < nbest || (np == nbest && sum < sbest)) {
                nbest = np;
                sbest = sum;
                std::copy(cur, cur + np, best);
            }
            return;
        }
        if (np + 1 > nbest || np == kMaxPasses) return;
        for (int r : {8, 6, 5, 4, 3, 2})
            if (r <= top && left % r == 0) {
                cur[np] = r;
                go(left / r, np + 1, sum + r, r);
            }
    };
    go(n, 0, 0, 8);
    auto twos = [](int r) { return r % 8 == 0 ? 3 : r % 4 == 0 ? 2 : r % 2 == 0 ? 1 : 0; };
    std::sort(best, best + nbest, [&](int a, int b) { return twos(a) != twos(b) ? twos(a) < twos(b) : a > b; });
    std::copy(best, best + nbest, rad);
    return nbest;
}

// ---- the batch's stages as kernels of their own, for the autotuner --------------
template <bool TW_LDS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
    batch_unit_kernel(const float2 *in, float2 *out, FftDesc f, XposeDesc d, int rw, int G)
{
    extern __shared__ __align__(16) unsigned char smem[];
    fft_xpose_unit<float2, -1, TW_LDS, kRadBatch, true, true>(in, out, f, d, rw, G, blockIdx.x, 1.f, false, smem);
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3)))
    batch_rows_kernel(const float2 *in, float2 *out, FftDesc f)
{
    extern __shared__ __align__(16) unsigned char smem[];
    fft_rows_block<float2, -1, kRadBatch>(in, out, f, blockIdx.x, 1.f, false, reinterpret_cast<float2 *>(smem));
}

template <int VU, int VV>
__global__ void __launch_bounds__(kThreads) batch_tile_kernel(const float2 *in, float2 *out, XposeDesc d)
{
    extern __shared__ __align__(16) unsigned char smem[];
    xpose_tile<float2, VU, VV>(in, out, d, blockIdx.x, smem);
}

hipError_t launch_batch_unit(const FftDesc &f, const XposeDesc &d, const void *in, void *out, hipStream_t s)
{
    int rw = 1, G = 1;
    fused_unit_shape(f.N, 8, d.Nv, d.nslices, 4096, &rw, &G);
    const bool tw = unit_tw_fits(f.N, 8);
    const dim3 grid((unsigned)(((d.Nv + rw - 1) / rw) * ((d.nslices + G - 1) / G)));
    auto kernel = tw ? &batch_unit_kernel<true> : &batch_unit_kernel<false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads),
                       fused_unit_bytes(f.N, rw, G, 8, tw), s, (const float2 *)in, (float2 *)out, f, d, rw, G);
    return hipGetLastError();
}

hipError_t launch_batch_rows(const FftDesc &f, const void *in, void *out, hipStream_t s)
{
    const dim3 grid((unsigned)((f.nrows + f.rows_per_wg - 1) / f.rows_per_wg));
    hipLaunchKernelGGL(batch_rows_kernel, grid, dim3(kThreads), (size_t)f.rows_per_wg * f.N * 8, s, (const float2 *)in,
                       (float2 *)out, f);
    return hipGetLastError();
}

// 16-byte accesses along even axes, as transpose stages choose them
int batch_xv(const XposeDesc &d)
{
    return ((d.Nu % 2 == 0 && d.TU >= 2) ? 1 : 0) | ((d.Nv % 2 == 0 && d.TV >= 2) ? 2 : 0);
}

hipError_t launch_batch_tile(const XposeDesc &d, const void *in, void *out, hipStream_t s)
{
    const int xv = batch_xv(d);
    auto kernel = xv == 3 ? &batch_tile_kernel<2, 2> : xv == 1 ? &batch_tile_kernel<2, 1>
                  : xv == 2 ? &batch_tile_kernel<1, 2> : &batch_tile_kernel<1, 1>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(d.tiles_u * d.tiles_v * d.tiles_g)), dim3(kThreads),
                       xpose_tile_bytes(d, 8) + 16, s, (const float2 *)in, (float2 *)out, d);
    return hipGetLastError();
}

namespace {

int batch_fail_hip(hipError_t e, const char *what)
{
    return fail(FFTRW_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

void batch_free(fft_batch_impl *b)
{
    if (!b) return;
    for (int d = 0; d < 2; ++d) {
        if (b->gexec[d]) (void)hipGraphExecDestroy(b->gexec[d]);
        if (b->graph[d]) (void)hipGraphDestroy(b->graph[d]);
    }
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    for (void *p : {(void *)b->d_items, (void *)b->d_tasks, (void *)b->d_ctr, (void *)b->d_level_task0,
                    (void *)b->d_level_units, (void *)b->d_timeouts})
        if (p) (void)hipFree(p);
    for (fft_plan_t p : b->plans) plan_free(p);
    delete b;
}

// enqueue reset + persistent kernel on stream s
int batch_enqueue(fft_batch_impl *b, int dir, hipStream_t s)
{
    const int64_t nctr = b->nctr;
    hipLaunchKernelGGL(batch_reset_kernel, dim3((unsigned)((nctr + 255) / 256)), dim3(256), 0, s, b->d_ctr, nctr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return batch_fail_hip(e, "batch reset launch");
    BatchLevelCtr *ctr = reinterpret_cast<BatchLevelCtr *>(b->d_ctr);
    const int nl = (int)b->level_units.size();
#define FFTRW_LAUNCH(D, T, L)                                                                                   \
    hipLaunchKernelGGL((batch_kernel<D, T, L>), dim3(b->grid), dim3(kThreads), b->lds, s, b->d_items, b->d_tasks, \
                       b->d_level_task0, b->d_level_units, nl, ctr, b->d_timeouts, b->wait_ticks)
    if (b->lean) {
        if (dir < 0) {
            if (b->tw_lds) FFTRW_LAUNCH(-1, true, true); else FFTRW_LAUNCH(-1, false, true);
        } else {
            if (b->tw_lds) FFTRW_LAUNCH(1, true, true); else FFTRW_LAUNCH(1, false, true);
        }
    } else {
        if (dir < 0) {
            if (b->tw_lds) FFTRW_LAUNCH(-1, true, false); else FFTRW_LAUNCH(-1, false, false);
        } else {
            if (b->tw_lds) FFTRW_LAUNCH(1, true, false); else FFTRW_LAUNCH(1, false, false);
        }
    }
#undef FFTRW_LAUNCH
    e = hipGetLastError();
    if (e != hipSuccess) return batch_fail_hip(e, "batch kernel launch");
    return FFTRW_OK;
}

}  // namespace
}  // namespace fftrw

struct fft_batch_s : fftrw::fft_batch_impl {};

using namespace fftrw;

extern "C" {

int fft_batch_plan(fft_batch_t *out, int n, const fft_item_desc *items, int precision, const char *tune_cache,
                   unsigned flags)
{
    g_last_error.clear();
    if (!out || !items || n < 1) return fail(FFTRW_E_ARG, "null output, null items or n < 1");
    TuneTable tune;
    const bool tuned = tune_cache && tune_load(tune_cache, tune_device_name(), fft_version(), &tune);
    *out = nullptr;
    if (precision != FFTRW_PREC_NATIVE)
        return fail(FFTRW_E_UNSUPPORTED, "the batched form runs the FP32 Stockham kernels");
    if (flags & ~(unsigned)(FFTRW_FLAG_COUNT_MOVED | FFTRW_FLAG_LEAVE_PERMUTED | FFTRW_FLAG_BATCH_NO_GRAPH |
                            FFTRW_FLAG_BATCH_NO_FUSE))
        return fail(FFTRW_E_UNSUPPORTED,
                    "the batched form supports COUNT_MOVED, LEAVE_PERMUTED, BATCH_NO_GRAPH and BATCH_NO_FUSE only");
    fft_batch_s *b = new (std::nothrow) fft_batch_s();
    if (!b) return fail(FFTRW_E_NOMEM, "out of host memory");
    b->n = n;
    b->flags = flags;
    // test hook: FFTRW_BATCH_WAIT_TICKS bounds each level wait (100 MHz
    // ticks) instead of 2 s, so tests can force the time-out path
    if (const char *w = std::getenv("FFTRW_BATCH_WAIT_TICKS")) b->wait_ticks = std::strtoull(w, nullptr, 10);
    const unsigned pflags = flags & (FFTRW_FLAG_COUNT_MOVED | FFTRW_FLAG_LEAVE_PERMUTED);
    const bool leave = (flags & FFTRW_FLAG_LEAVE_PERMUTED) != 0;
    b->h_items.resize(n);
    size_t lds = 16, lds_tw = 16;  // LDS per group without and with staged twiddles
    bool tw_fits = true;          // every fused step's table fits (unit_tw_fits)
    int max_stage = 0;
    std::vector<char> listed((size_t)n * kMaxDims, 0);  // the step's radices are the cache's
    for (int i = 0; i < n; ++i) {
        const fft_item_desc &it = items[i];
        fft_plan_t p = nullptr;
        int rc = plan_create(&p, it.M, it.dims, it.P, it.has_order ? it.order : nullptr, FFTRW_C64,
                             FFTRW_PREC_NATIVE, pflags, true, tuned ? &tune : nullptr, nullptr);
        if (rc) {
            std::string m = "item " + std::to_string(i) + ": " + g_last_error;
            batch_free(b);
            return fail(rc, m);
        }
        b->plans.push_back(p);
        BatchItemDev &d = b->h_items[i];
        std::memset(&d, 0, sizeof(d));
        d.M = it.M;
        const int nx = leave ? it.M - 1 : it.M;
        d.nx = nx;
        d.buf[2] = (float2 *)p->work;
        d.inv_scale = (float)(1.0 / (double)p->T);
        for (int t = 0; tuned && t < it.M; ++t) {
            auto rt = tune.rows.find(p->fft[t].N);
            listed[(size_t)i * kMaxDims + t] = rt != tune.rows.end() && valid_radices(rt->second.radix, p->fft[t].N);
        }
        int64_t units = 0;
        // fused schedule: a unit's shape is fused_unit_shape's
        d.fused = !(flags & FFTRW_FLAG_BATCH_NO_FUSE);
        if (d.fused) {
            d.nstage = it.M;
            int cur = 0;
            for (int t = 0; t < it.M; ++t) {
                d.prefix[t] = units;
                d.fft[t] = p->fft[t];
                if (t < nx) {
                    d.xp[t] = p->xp[t];
                    const int N = d.fft[t].N;
                    if (tuned) {
                        // the radix order the autotuner timed in the fused unit
                        // (it differs from the separate row kernel's), checked
                        // as the plan checks the row kernel's
                        auto ft = tune.fused.find({N, (int)d.xp[t].Nv});
                        if (ft != tune.fused.end()) {
                            const std::vector<int> &rad = ft->second;
                            if (valid_radices(rad, N)) {
                                d.fft[t].npass = (int)rad.size();
                                for (int q = 0; q < d.fft[t].npass; ++q) d.fft[t].radix[q] = rad[q];
                                listed[(size_t)i * kMaxDims + t] = 1;
                            }
                        }
                    }
                    int rw = 1, G = 1;
                    fused_unit_shape(N, 8, d.xp[t].Nv, d.xp[t].nslices, 4096, &rw, &G);
                    d.frw[t] = rw;
                    d.fg[t] = G;
                    d.src[t] = t == 0 ? 0 : cur;
                    d.dst[t] = ((nx - 1 - t) % 2 == 0) ? 1 : 2;
                    cur = d.dst[t];
                    units += ((d.xp[t].Nv + rw - 1) / rw) * ((d.xp[t].nslices + G - 1) / G);
                    lds = std::max(lds, fused_unit_bytes(N, rw, G, 8, false));
                    lds_tw = std::max(lds_tw, fused_unit_bytes(N, rw, G, 8, true));
                    tw_fits = tw_fits && unit_tw_fits(N, 8);
                } else {
                    // LEAVE_PERMUTED: the last FFT step runs in place on the output
                    d.src[t] = 1;
                    d.dst[t] = 1;
                    units += (d.fft[t].nrows + d.fft[t].rows_per_wg - 1) / d.fft[t].rows_per_wg;
                    lds = std::max(lds, (size_t)d.fft[t].rows_per_wg * d.fft[t].N * 8);
                }
            }
            d.prefix[d.nstage] = units;
            max_stage = std::max(max_stage, d.nstage);
            b->any_fused = true;
            continue;
        }
        d.nstage = it.M + nx;
        // buffer sequence of the pipeline: FFT 0 reads the input; transposes alternate
        const int b0 = (nx % 2 == 0) ? 1 : 2, b1 = b0 == 1 ? 2 : 1;
        int cur = b0, other = b1;
        for (int st = 0; st < d.nstage; ++st) {
            d.prefix[st] = units;
            const int t = st >> 1;
            if ((st & 1) == 0) {
                d.src[st] = t == 0 ? 0 : cur;
                d.dst[st] = cur;
                d.fft[t] = p->fft[t];
                units += (d.fft[t].nrows + d.fft[t].rows_per_wg - 1) / d.fft[t].rows_per_wg;
                lds = std::max(lds, (size_t)d.fft[t].rows_per_wg * d.fft[t].N * 8);
            } else {
                d.src[st] = cur;
                d.dst[st] = other;
                std::swap(cur, other);
                d.xp[t] = p->xp[t];
                d.xv[t] = batch_xv(d.xp[t]);
                units += d.xp[t].tiles_u * d.xp[t].tiles_v * d.xp[t].tiles_g;
                lds = std::max(lds, xpose_tile_bytes(d.xp[t], 8) + 16);
            }
        }
        d.prefix[d.nstage] = units;
        max_stage = std::max(max_stage, d.nstage);
    }
    // stage level by stage level, items in order; units numbered within a level
    for (int s = 0; s < max_stage; ++s) {
        b->level_task0.push_back((int)b->h_tasks.size());
        int64_t lvl = 0;
        for (int i = 0; i < n; ++i) {
            const BatchItemDev &d = b->h_items[i];
            if (s >= d.nstage) continue;
            const int64_t cnt = d.prefix[s + 1] - d.prefix[s];
            if (cnt <= 0) continue;
            b->h_tasks.push_back({i, s, lvl, cnt});
            lvl += cnt;
        }
        // claims count in 32 bits (see claim); every group claims at most
        // once past the end of a level
        if (lvl >= (int64_t{1} << 31)) {
            batch_free(b);
            return fail(FFTRW_E_SIZE, "a stage level of the batch has 2^31 or more units");
        }
        b->level_units.push_back(lvl);
        b->total += lvl;
    }
    b->level_task0.push_back((int)b->h_tasks.size());
    // twiddles in LDS when every fused step's table fits; the groups of the
    // separate stages need no more LDS either way
    b->tw_lds = b->any_fused && tw_fits;
    b->lds = (std::max(lds, b->tw_lds ? lds_tw : (size_t)0) + 15) & ~(size_t)15;
    // Every FFT step of a batch runs radices 2 to 6 and 8 only (16 becomes
    // 4 x 4, in place), in the fused and the separate schedules alike so that
    // the two stay bit-identical.  When every stage is a fused unit (no
    // LEAVE_PERMUTED, no BATCH_NO_FUSE) the batch then runs batch_kernel's
    // LEAN form: without the separate stage kernels and the larger passes it
    // holds four waves per SIMD instead of three (256 uneven items 5.95 -> 5.33 ms when
    // it was introduced).
    b->lean = !(flags & (FFTRW_FLAG_LEAVE_PERMUTED | FFTRW_FLAG_BATCH_NO_FUSE));
    for (fft_plan_t p : b->plans)
        if (p->T * (int64_t)sizeof(float2) >= (int64_t{1} << 32)) b->lean = false;  // 32-bit offsets
    for (int i = 0; i < n; ++i) {
        BatchItemDev &d = b->h_items[i];
        for (int t = 0; t < d.M; ++t) {
            FftDesc &f = d.fft[t];
            int rad[kMaxPasses], np = 0;
            int def[kMaxPasses];
            if (!listed[(size_t)i * kMaxDims + t] ||
                (!tune.batch_lists && f.npass == factor_radices(f.N, def) && std::equal(def, def + f.npass, f.radix))) {
                f.npass = batch_radices(f.N, f.radix);
                continue;
            }
            // (rows hold at most 4096 = 2^kMaxPasses points, so any list fits)
            for (int q = 0; q < f.npass; ++q) {
                if (f.radix[q] == 16) {
                    rad[np++] = 4;
                    rad[np++] = 4;
                } else {
                    rad[np++] = f.radix[q];
                }
            }
            f.npass = np;
            for (int q = 0; q < np; ++q) f.radix[q] = rad[q];
        }
    }
    b->moved_off.resize(n);
    b->nctr = (int64_t)(b->level_units.size() * sizeof(BatchLevelCtr) / sizeof(unsigned long long));
    for (int i = 0; i < n; ++i) {
        b->moved_off[i] = b->nctr;
        b->nctr += (int64_t)b->h_items[i].M * kCountBlock;
    }
    int dev = 0, ncu = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu,
            b->lean ? (b->tw_lds ? batch_kernel<-1, true, true> : batch_kernel<-1, false, true>)
                    : (b->tw_lds ? batch_kernel<-1, true, false> : batch_kernel<-1, false, false>),
            kThreads, b->lds);
    if (e != hipSuccess || per_cu < 1 || ncu < 1) {
        batch_free(b);
        return e != hipSuccess ? batch_fail_hip(e, "occupancy query") : fail(FFTRW_E_DEVICE, "kernel does not fit");
    }
    // no more groups than a level has units: every group claims past its end.
    // The general kernel takes no more than the largest level's rounds need
    // either, as its levels are many and each costs every group its end
    // (sixteen 64^3 with BATCH_NO_FUSE, 1024 units a level: 220 us on 768
    // groups, 180 on 512)
    const int64_t most = *std::max_element(b->level_units.begin(), b->level_units.end());
    int64_t groups = std::min<int64_t>((int64_t)per_cu * ncu, most);
    if (!b->lean && groups > 0) {
        const int64_t rounds = (most + groups - 1) / groups;
        groups = (most + rounds - 1) / rounds;
    }
    b->grid = (int)groups;
    e = hipMalloc(&b->d_items, sizeof(BatchItemDev) * (size_t)n);
    if (e == hipSuccess) e = hipMalloc(&b->d_tasks, sizeof(BatchTask) * b->h_tasks.size());
    if (e == hipSuccess) e = hipMalloc(&b->d_ctr, sizeof(unsigned long long) * (size_t)b->nctr);
    if (e == hipSuccess) e = hipMalloc(&b->d_timeouts, sizeof(unsigned long long));
    if (e == hipSuccess) e = hipMemset(b->d_timeouts, 0, sizeof(unsigned long long));
    if (e == hipSuccess && (flags & FFTRW_FLAG_COUNT_MOVED)) {
        // owner-change counters of every transpose live in the batch's counter
        // block, which the graph's reset kernel clears before each launch
        for (int i = 0; i < n; ++i)
            for (int t = 0; t < b->h_items[i].M; ++t)
                if (b->h_items[i].xp[t].count)
                    b->h_items[i].xp[t].counter = b->d_ctr + b->moved_off[i] + (int64_t)t * kCountBlock;
    }
    if (e == hipSuccess)
        e = hipMemcpy(b->d_tasks, b->h_tasks.data(), sizeof(BatchTask) * b->h_tasks.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMalloc(&b->d_level_task0, sizeof(int) * b->level_task0.size());
    if (e == hipSuccess) e = hipMalloc(&b->d_level_units, sizeof(int64_t) * b->level_units.size());
    if (e == hipSuccess)
        e = hipMemcpy(b->d_level_task0, b->level_task0.data(), sizeof(int) * b->level_task0.size(),
                      hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(b->d_level_units, b->level_units.data(), sizeof(int64_t) * b->level_units.size(),
                      hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        batch_free(b);
        return fail(FFTRW_E_NOMEM, "device allocation for the batch failed");
    }
    b->tuned = tuned;
    int64_t units = 0;
    for (int64_t u : b->level_units) units += u;
    log_line(1, "batch of %d items: %lld units in %zu stage levels, %d resident groups, %s stages%s%s", n,
             (long long)units, b->level_units.size(), b->grid, b->any_fused ? "fused" : "separate",
             b->lean ? " (lean kernel: fused units of radices 2 to 6 and 8)" : "", tuned ? ", tuned" : "");
    *out = b;
    return FFTRW_OK;
}

static int batch_exec(fft_batch_t b, void *const *in, void *const *out, void *stream, int dir)
{
    g_last_error.clear();
    if (!b || !in || !out) return fail(FFTRW_E_ARG, "null batch or pointer arrays");
    if (b->timed_out)
        return fail(FFTRW_E_DEVICE, "an earlier launch of this batch timed out at a level barrier");
    bool changed = !b->pointers_set;
    for (int i = 0; i < b->n; ++i) {
        if (!in[i] || !out[i]) return fail(FFTRW_E_ARG, "null buffer for item " + std::to_string(i));
        if (b->h_items[i].fused && in[i] == out[i])
            return fail(FFTRW_E_ARG, "item " + std::to_string(i) +
                                         ": fused stages need in != out (plan with FFTRW_FLAG_BATCH_NO_FUSE for in place)");
        BatchItemDev &d = b->h_items[i];
        if (d.buf[0] != in[i] || d.buf[1] != out[i]) changed = true;
        d.buf[0] = (float2 *)in[i];
        d.buf[1] = (float2 *)out[i];
    }
    hipStream_t s = (hipStream_t)stream;
    if (changed) {
        // the item table is read by the kernel; update it in stream order
        hipError_t e = hipStreamSynchronize(s);
        if (e == hipSuccess)
            e = hipMemcpy(b->d_items, b->h_items.data(), sizeof(BatchItemDev) * (size_t)b->n, hipMemcpyHostToDevice);
        if (e != hipSuccess) return batch_fail_hip(e, "item table update");
        b->pointers_set = true;
    }
    if (b->flags & FFTRW_FLAG_BATCH_NO_GRAPH) return batch_enqueue(b, dir, s);
    const int di = dir < 0 ? 0 : 1;
    if (!b->gexec[di]) {
        hipError_t e = hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return batch_fail_hip(e, "graph capture begin");
        int rc = batch_enqueue(b, dir, b->cap_stream);
        e = hipStreamEndCapture(b->cap_stream, &b->graph[di]);
        if (rc) return rc;
        if (e != hipSuccess) return batch_fail_hip(e, "graph capture end");
        e = hipGraphInstantiate(&b->gexec[di], b->graph[di], nullptr, nullptr, 0);
        if (e != hipSuccess) return batch_fail_hip(e, "graph instantiate");
    }
    hipError_t e = hipGraphLaunch(b->gexec[di], s);
    if (e != hipSuccess) return batch_fail_hip(e, "graph launch");
    return FFTRW_OK;
}

int fft_batch_exec_fwd(fft_batch_t b, void *const *in, void *const *out, void *stream)
{
    return batch_exec(b, in, out, stream, -1);
}

int fft_batch_exec_inv(fft_batch_t b, void *const *in, void *const *out, void *stream)
{
    return batch_exec(b, in, out, stream, 1);
}

int fft_batch_stats(fft_batch_t b, int64_t *moved, int64_t *analytic, int64_t *units, int *error)
{
    g_last_error.clear();
    if (!b) return fail(FFTRW_E_ARG, "null batch");
    if (units) *units = b->total;
    std::vector<unsigned long long> h((size_t)b->nctr, 0ull);
    unsigned long long timeouts = 0;
    {
        hipError_t e = hipDeviceSynchronize();
        if (e == hipSuccess && moved)
            e = hipMemcpy(h.data(), b->d_ctr, sizeof(unsigned long long) * h.size(), hipMemcpyDeviceToHost);
        if (e == hipSuccess) e = hipMemcpy(&timeouts, b->d_timeouts, sizeof(timeouts), hipMemcpyDeviceToHost);
        if (e != hipSuccess) return batch_fail_hip(e, "reading batch counters");
    }
    const bool leave = (b->flags & FFTRW_FLAG_LEAVE_PERMUTED) != 0;
    const bool counted = (b->flags & FFTRW_FLAG_COUNT_MOVED) != 0;
    int off = 0;
    for (int i = 0; i < b->n; ++i) {
        const int M = b->h_items[i].M;
        for (int t = 0; t < M; ++t) {
            if (analytic) analytic[off + t] = b->plans[i]->analytic[t];
            if (moved) {
                int64_t sum = -1;
                if (counted && !(leave && t == M - 1)) {
                    sum = 0;
                    for (int k = 0; k < kCountSlots; ++k)
                        sum += (int64_t)h[b->moved_off[i] + (int64_t)t * kCountBlock + (int64_t)k * kCountStride];
                }
                moved[off + t] = sum;
            }
        }
        off += M;
    }
    if (error) *error = (int)std::min<unsigned long long>(timeouts, 0x7fffffffull);
    if (timeouts) {
        b->timed_out = true;
        return fail(FFTRW_E_DEVICE, std::to_string(timeouts) +
                                        " level-barrier wait(s) timed out; results of this batch are unreliable");
    }
    return FFTRW_OK;
}

int fft_batch_destroy(fft_batch_t b)
{
    g_last_error.clear();
    batch_free(b);
    return FFTRW_OK;
}

}  // extern "C"
