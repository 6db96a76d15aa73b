// fft_ct.hip -- instances of the compile-time row FFT kernels (fft_ct.hpp) for
// the lengths of one share of the table.  The file is compiled FFTRW_CT_PARTS
// times, with FFTRW_CT_PART = 0 .. FFTRW_CT_PARTS - 1, so that the instances
// build in parallel.
#include <hip/hip_runtime.h>

#include "fft_ct.hpp"

namespace fftrw {

namespace {

template <class P, int p> constexpr int tw_count()
{
    return CtPass<P, p>::tw_off + (p > 0 ? CtPass<P, p>::Ns * (CtPass<P, p>::R - 1) : 0);
}

template <typename C, int N> CtEntry entry()
{
    using P = CtPlan<C, N>;
    CtEntry e{};
    e.N = N;
    e.esz = (int)sizeof(C);
    e.L = P::L;
    e.np = P::NP;
    for (int i = 0; i < P::NP; ++i) e.r[i] = P::c.r[i];
    e.tw_count = tw_count<P, P::NP - 1>();
    // (rows that pass through LDS take the threads of CtStage)
    e.min_threads = P::DIRECT && P::STORE_DIRECT ? 64 : 1 << CtStage<P, C>::LW;
    if (e.min_threads < 64) e.min_threads = 64;
    if (e.min_threads < P::L) e.min_threads = P::L;
    static_assert((1 << CtStage<P, C>::LW) <= P::MAXNT || (P::DIRECT && P::STORE_DIRECT), "a row's threads fit a group");
    e.max_threads = P::MAXNT;
    e.pitch = ct_row_pitch<P>();
    e.staged = !P::DIRECT;
    e.fused = &ct_fused_kernel<C, N>;
    e.rows = &ct_rows_kernel<C, P, false>;
    if constexpr (N * sizeof(C) % 128 != 0) e.rows_block = &ct_rows_kernel<C, P, true>;
    if constexpr (!P::DIRECT || !P::STORE_DIRECT) e.rows_straight = &ct_rows_kernel<C, CtStraight<C, N>, false>;
    return e;
}

template <int I> void add(CtEntry *out, int &n)
{
    if constexpr (I < kCtLengths) {
        if constexpr (I % FFTRW_CT_PARTS == FFTRW_CT_PART) {
            out[n++] = entry<float2, ct_length(I)>();
            if constexpr (ct_length(I) <= kCtMaxFp64) out[n++] = entry<double2, ct_length(I)>();
        }
        add<I + 1>(out, n);
    }
}

}  // namespace

#define FFTRW_CT_NAME2(p) ct_part_##p
#define FFTRW_CT_NAME(p) FFTRW_CT_NAME2(p)
int FFTRW_CT_NAME(FFTRW_CT_PART)(CtEntry *out)
{
    int n = 0;
    add<0>(out, n);
    return n;
}

}  // namespace fftrw
