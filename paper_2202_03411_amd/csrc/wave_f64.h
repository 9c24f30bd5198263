// FP64 lane operations and the FP64 matrix instruction (device code only).
#pragma once

#include <hip/hip_runtime.h>

namespace msft {

// One DPP step on an FP64 value (both 32-bit halves moved by the same lane pattern;
// lanes outside the row mask, or whose source lies outside their row, read 0).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROW_MASK, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROW_MASK, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | (unsigned long long)lo));
}

// Inclusive prefix sum over each row of 16 lanes (row_shr 1, 2, 4, 8).
__device__ __forceinline__ double row_prefix_f64(double v)
{
    v += dpp_f64<0x111, 0xF>(v);
    v += dpp_f64<0x112, 0xF>(v);
    v += dpp_f64<0x114, 0xF>(v);
    v += dpp_f64<0x118, 0xF>(v);
    return v;
}

// Lane 15's value of each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ double row_last_f64(double v) { return __shfl(v, 15, 16); }

// v_mfma_f64_16x16x4_f64: D (16 x 16) += A (16 x 4) B (4 x 16).  Lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and, in element r, D[4 r + l / 16][l % 16].
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// f(0) ... f(steps - 1), U at a time so that the loads of several steps are in flight.
template <int U, typename F>
__device__ __forceinline__ void for_steps(int steps, F f)
{
    int k = 0;
    for (; k + U <= steps; k += U)
#pragma unroll
        for (int u = 0; u < U; ++u) f(k + u);
    for (; k < steps; ++k) f(k);
}

}  // namespace msft
