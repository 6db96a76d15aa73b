// fft_rows.hip -- the FP64-generated twiddle tables w_N^e of the run-time-radix
// kernels, and the launches of those that plans still reach: rows of complex128
// past the compile-time kernels (2049 to 4096 points) and steps of single
// points.  The fused unit's shape rule exported for tests
// (fft_fused_unit_shape).
#include <hip/hip_runtime.h>

#include "../../include/fftrw.h"
#include "errors.hpp"
#include "fft_generic.hpp"
#include "fused_generic.hpp"

namespace fftrw {

// ---- twiddle table: w_N^e = exp(-2 pi i e / N), computed in FP64 -------------
template <typename C>
__global__ void __launch_bounds__(kThreads) twiddle_kernel(C *out, int64_t n)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    double s, c;
    unit_root((int)e, (int)n, &c, &s);
    out[e] = mk<C>((typename RealOf<C>::type)c, (typename RealOf<C>::type)s);
}

hipError_t launch_twiddles(void *out, int64_t n, bool fp64, hipStream_t s)
{
    dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
    if (fp64)
        hipLaunchKernelGGL(twiddle_kernel<double2>, grid, dim3(kThreads), 0, s, (double2 *)out, n);
    else
        hipLaunchKernelGGL(twiddle_kernel<float2>, grid, dim3(kThreads), 0, s, (float2 *)out, n);
    return hipGetLastError();
}

template <typename C, int DIR, bool LEAN>
__global__ void __launch_bounds__(kThreads)
    fft_rows_kernel(const C *in, C *out, FftDesc d, typename RealOf<C>::type scale, int do_scale)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    fft_rows_block<C, DIR, LEAN ? kRadSmall : kRadRows>(in, out, d, blockIdx.x, scale, do_scale != 0,
                                                        reinterpret_cast<C *>(smem_raw));
}

// Radix lists without 8 and 16 (lengths with at most two factors 2) run the
// kernel compiled for radices 2 to 5 only.
bool lean_radices(const FftDesc &d)
{
    for (int q = 0; q < d.npass; ++q)
        if (d.radix[q] == 8 || d.radix[q] == 16) return false;
    return true;
}

hipError_t launch_fft_rows(const FftDesc &d, bool fp64, int dir, const void *in, void *out, double scale,
                           hipStream_t s)
{
    const int64_t nblk = (d.nrows + d.rows_per_wg - 1) / d.rows_per_wg;
    if (nblk <= 0) return hipSuccess;
    const size_t lds = (size_t)d.rows_per_wg * d.N * (fp64 ? 16 : 8);
    const int do_scale = scale != 1.0;
    dim3 grid((unsigned)nblk), block(kThreads);
#define FFTRW_LAUNCH(C, D, L, SC) \
    hipLaunchKernelGGL((fft_rows_kernel<C, D, L>), grid, block, lds, s, (const C *)in, (C *)out, d, SC, do_scale)
    if (d.N == 1) {  // scaled copies: no direction
        if (fp64) FFTRW_LAUNCH(double2, -1, true, scale); else FFTRW_LAUNCH(float2, -1, true, (float)scale);
    } else if (!fp64) {
        return hipErrorInvalidValue;  // compile-time kernels
    } else if (lean_radices(d)) {
        if (dir < 0) FFTRW_LAUNCH(double2, -1, true, scale); else FFTRW_LAUNCH(double2, 1, true, scale);
    } else {
        if (dir < 0) FFTRW_LAUNCH(double2, -1, false, scale); else FFTRW_LAUNCH(double2, 1, false, scale);
    }
#undef FFTRW_LAUNCH
    return hipGetLastError();
}

template <typename C>
__global__ void __launch_bounds__(kThreads)
    xpose_points_kernel(const C *in, C *out, FftDesc f, XposeDesc d, int rw, int G, typename RealOf<C>::type scale,
                        int do_scale)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    fft_xpose_unit<C, -1, true, kRadSmall>(in, out, f, d, rw, G, blockIdx.x, scale, do_scale != 0, smem_raw);
}

// a step of single points fused with the transpose that follows
hipError_t launch_xpose_points(const FftDesc &f, const XposeDesc &d, bool fp64, const void *in, void *out, double scale,
                               hipStream_t s)
{
    if (f.N != 1) return hipErrorInvalidValue;
    const size_t esz = fp64 ? 16 : 8;
    int rw = 1, G = 1;
    fused_unit_shape(f.N, esz, d.Nv, d.nslices, fp64 ? 2048 : 4096, &rw, &G);
    const int64_t nblk = ((d.Nv + rw - 1) / rw) * ((d.nslices + G - 1) / G);
    if (nblk <= 0) return hipSuccess;
    if (nblk >= (int64_t)0x7fffffff) return hipErrorInvalidValue;
    const size_t lds = fused_unit_bytes(f.N, rw, G, esz, true);
    const int do_scale = scale != 1.0;
    dim3 grid((unsigned)nblk), block(kThreads);
    if (fp64)
        hipLaunchKernelGGL(xpose_points_kernel<double2>, grid, block, lds, s, (const double2 *)in, (double2 *)out, f, d, rw,
                           G, scale, do_scale);
    else
        hipLaunchKernelGGL(xpose_points_kernel<float2>, grid, block, lds, s, (const float2 *)in, (float2 *)out, f, d, rw, G,
                           (float)scale, do_scale);
    return hipGetLastError();
}

}  // namespace fftrw

extern "C" int fft_fused_unit_shape(int N, int esz, int64_t Nv, int64_t nslices, int *rw, int *G)
{
    fftrw::g_last_error.clear();
    if (N < 2 || Nv < 1 || nslices < 1 || (esz != 8 && esz != 16) || !rw || !G)
        return fftrw::fail(FFTRW_E_ARG, "fft_fused_unit_shape: N >= 2, Nv >= 1, nslices >= 1, esz 8 or 16, "
                                        "non-null outputs");
    fftrw::fused_unit_shape(N, (size_t)esz, Nv, nslices, esz == 16 ? 2048 : 4096, rw, G);
    return FFTRW_OK;
}
