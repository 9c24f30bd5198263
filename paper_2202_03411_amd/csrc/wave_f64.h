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

// The same over groups of L = 16 or 32 lanes.
template <int L>
__device__ __forceinline__ double group_prefix_f64(double v)
{
    v = row_prefix_f64(v);
    if (L == 32) v += dpp_f64<0x142, 0xA>(v);   // lane 15 of rows 0 and 2 into rows 1 and 3
    return v;
}
template <int L>
__device__ __forceinline__ double group_last_f64(double v) { return __shfl(v, L - 1, L); }

// v_mfma_f64_16x16x4_f64: D (16 x 16) += A (16 x 4) B (4 x 16).  Lane l holds
// A[l % 16][l / 16], B[l / 16][l % 16] and, in element r, D[4 r + l / 16][l % 16].
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// v_mfma_f64_4x4x4_4b_f64: four independent 4 x 4 x 4 products.  Lane l belongs to block
// (l / 4) % 4 and holds A[l % 4][l / 16], B[l / 16][l % 4] and D[l / 16][l % 4] of it.
__device__ __forceinline__ double mfma_f64_4b(double a, double b, double c)
{
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// A table pointer that was itself read from memory: without the address space the
// compiler emits flat loads, which also wait for the LDS.
template <typename T>
__device__ __forceinline__ const T __attribute__((address_space(1))) * as_global(const T* p)
{
    return (const T __attribute__((address_space(1)))*)p;
}
template <typename T>
__device__ __forceinline__ T __attribute__((address_space(1))) * as_global(T* p)
{
    return (T __attribute__((address_space(1)))*)p;
}
typedef const double __attribute__((address_space(1))) * gcdouble;
typedef double __attribute__((address_space(1))) * gdouble;

// A double at a wave-uniform address plus a lane's byte offset: one load with a scalar
// base, the address arithmetic of a loop staying on the scalar unit.
__device__ __forceinline__ double load_at(gcdouble base, uint32_t offset)
{
    return *(gcdouble)((const char __attribute__((address_space(1)))*)base + offset);
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

// Operands of a product's steps: step k of a stream is at p + k inc (wave-uniform), the
// lane's byte offset added.
struct Stream {
    gcdouble p;
    int64_t inc;
    uint32_t off;
};

// comp(k, x) for k = 0 ... steps - 1, x[i] the operand of stream i.  The loads of U steps
// are issued before the first of their products (left to itself the compiler places each
// load next to its use and waits for it there).
template <int U, int NS, typename C>
__device__ __forceinline__ void staged(const Stream (&s)[NS], int steps, C comp)
{
    gcdouble p[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) p[i] = s[i].p;
    int k = 0;
    for (; k + U <= steps; k += U) {
        double x[U][NS];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NS; ++i) x[u][i] = load_at(p[i] + u * s[i].inc, s[i].off);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) comp(k + u, x[u]);
#pragma unroll
        for (int i = 0; i < NS; ++i) p[i] += U * s[i].inc;
    }
    if (U > 1 && k < steps) {
        double x[U][NS];
#pragma unroll
        for (int u = 0; u + 1 < U; ++u) {
            const int v = min(u, steps - 1 - k);
#pragma unroll
            for (int i = 0; i < NS; ++i) x[u][i] = load_at(p[i] + v * s[i].inc, s[i].off);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u + 1 < U; ++u)
            if (k + u < steps) comp(k + u, x[u]);
    }
}

// The wave's index in its workgroup, as a scalar.
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

constexpr f64x4 F64X4_ZERO = {0.0, 0.0, 0.0, 0.0};

// Four waves' partial sums of four product tiles: wave w gets tile w's total, the others'
// parts of it through LDS.
constexpr int SUM_WAVES_LDS = 4 * 3 * 4 * 64;
__device__ __forceinline__ f64x4 sum_waves(double* red, const f64x4* t, int wave, int lane)
{
    f64x4 own = F64X4_ZERO;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k == wave) {
            own = t[k];
            continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) red[((k * 3 + (wave < k ? wave : wave - 1)) * 4 + r) * 64 + lane] = t[k][r];
    }
    __syncthreads();
    f64x4 s = F64X4_ZERO;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w == wave) {
            s += own;
            continue;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] += red[((wave * 3 + (w < wave ? w : w - 1)) * 4 + r) * 64 + lane];
    }
    return s;
}

// exp(-k0 dz (b + i d)) of one slice by its Taylor series, exponents below 1/8: six and
// three terms (remainders below 4e-10).
__device__ __forceinline__ void slice_factor(double x, double y, double* er, double* ei)
{
    const double q = y * y;
    double m = 1.0 / 720.0;
    m = __builtin_fma(m, x, 1.0 / 120.0);
    m = __builtin_fma(m, x, 1.0 / 24.0);
    m = __builtin_fma(m, x, 1.0 / 6.0);
    m = __builtin_fma(m, x, 0.5);
    m = __builtin_fma(m, x, 1.0);
    m = __builtin_fma(m, x, 1.0);
    double c = __builtin_fma(q, -1.0 / 720.0, 1.0 / 24.0);
    c = __builtin_fma(__builtin_fma(c, q, -0.5), q, 1.0);
    double s = __builtin_fma(q, 1.0 / 120.0, -1.0 / 6.0);
    s = __builtin_fma(s * q, y, y);
    *er = m * c;
    *ei = m * s;
}

// exp, sin and cos for the transmission, in FP64 arithmetic (the FP32 rate on this chip)
// to about 1e-9, far below the FP32 results: range reduction and Taylor series on what is
// left, exp over |r| <= ln(2) / 2 to r^8 / 8!, sin and cos over |r| <= pi / 4 to r^9 / 9!
// and r^10 / 10! (remainders below 3e-9).
__device__ __forceinline__ double exp_series(double r)
{
    double p = 1.0 / 40320.0;
    p = __builtin_fma(p, r, 1.0 / 5040.0);
    p = __builtin_fma(p, r, 1.0 / 720.0);
    p = __builtin_fma(p, r, 1.0 / 120.0);
    p = __builtin_fma(p, r, 1.0 / 24.0);
    p = __builtin_fma(p, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    return __builtin_fma(p, r, 1.0);
}

__device__ __forceinline__ double exp_reduced(double x)
{
    const double n = rint(x * 1.4426950408889634074);
    return __builtin_ldexp(exp_series(__builtin_fma(n, -0.69314718055994530942, x)), (int)n);
}

__device__ __forceinline__ void sincos_reduced(double x, double* sn, double* cs)
{
    const double n = rint(x * 0.63661977236758134308);
    const double r = __builtin_fma(n, -1.5707963267948966192, x), q = r * r;
    double s = 1.0 / 362880.0, c = -1.0 / 3628800.0;
    s = __builtin_fma(s, q, -1.0 / 5040.0);
    s = __builtin_fma(s, q, 1.0 / 120.0);
    s = __builtin_fma(s, q, -1.0 / 6.0);
    s = __builtin_fma(s * q, r, r);
    c = __builtin_fma(c, q, 1.0 / 40320.0);
    c = __builtin_fma(c, q, -1.0 / 720.0);
    c = __builtin_fma(c, q, 1.0 / 24.0);
    c = __builtin_fma(c, q, -0.5);
    c = __builtin_fma(c, q, 1.0);
    // the quadrant from the fraction of n / 4, exact for any n
    const double f = n * 0.25;
    const int k = (int)(4.0 * (f - floor(f)));
    const double a = k & 1 ? c : s, b = k & 1 ? s : c;
    *sn = k & 2 ? -a : a;
    *cs = (k + 1) & 2 ? -b : b;
}

// dV exp(-i qc z) T along a lane's slices, T = exp(-k0 dz S) (1 without MSFT).  In full at
// the first slice, (Sb, Sd) the sums of beta and delta before it and (rr, ri) the table's
// dV exp(-i qc z) there, then multiplied by each slice's own factor and the rotation's step
// exp(-i qc dz).  A wave that holds a factor's exponent of 1/8 or more evaluates T in full
// at every slice.
template <bool MSFT>
struct Propagator {
    double Sb, Sd, k0dz, rr, ri, cr, ci, tr, ti;
    bool small;

    __device__ __forceinline__ void full()
    {
        double sn, cs;
        const double m = exp_reduced(-k0dz * Sb);
        sincos_reduced(-k0dz * Sd, &sn, &cs);
        sn *= m;
        cs *= m;
        tr = cs * rr - sn * ri;
        ti = cs * ri + sn * rr;
    }
    template <int K>
    __device__ __forceinline__ void start(double sb, double sd, const float* b, const float* d, double k, double r0,
                                          double r1, double step_r, double step_i)
    {
        rr = tr = r0;
        ri = ti = r1;
        cr = step_r;
        ci = step_i;
        if (!MSFT) return;
        float big = 0.0f;
#pragma unroll
        for (int e = 0; e + 1 < K; ++e) big = fmaxf(big, fmaxf(fabsf(b[e]), fabsf(d[e])));
        Sb = sb;
        Sd = sd;
        k0dz = k;
        small = __all(k * (double)big < 0.125);
        full();
    }
    // To the slice after one of (b, d); SMALL is `small`, taken out of the callers' loops.
    template <bool SMALL>
    __device__ __forceinline__ void next(double b, double d)
    {
        if (MSFT && SMALL) {
            double er, ei;
            slice_factor(-k0dz * b, -k0dz * d, &er, &ei);
            const double fr = er * cr - ei * ci, fi = er * ci + ei * cr, t = tr;
            tr = t * fr - ti * fi;
            ti = t * fi + ti * fr;
            return;
        }
        const double t = rr;
        rr = t * cr - ri * ci;
        ri = t * ci + ri * cr;
        if (MSFT) {
            Sb += b;
            Sd += d;
            full();
            __builtin_amdgcn_sched_barrier(0);   // one slice at a time: the registers are the common case's
        } else {
            tr = rr;
            ti = ri;
        }
    }
};

// K slices of a column from z on, zero past its end, in 16-byte (8-byte) pieces where the
// column's rows are aligned to them.  Every lane loads (past the end, the column's last
// piece), so that no load waits behind a branch.
template <int K>
__device__ __forceinline__ void load_slices(const float* dc, const float* bc, int z, int nz, bool in, float* d,
                                            float* b)
{
    if ((nz & 3) == 0) {
        if (K % 4 == 0) {
            float4 dv[K / 4 + 1], bv[K / 4 + 1];
#pragma unroll
            for (int k = 0; k + 3 < K; k += 4) {
                const int at = min(z + k, nz - 4);
                dv[k / 4] = *(const float4*)(dc + at);
                bv[k / 4] = *(const float4*)(bc + at);
            }
#pragma unroll
            for (int k = 0; k + 3 < K; k += 4) {
                const bool ok = in && z + k < nz;
                d[k] = ok ? dv[k / 4].x : 0.0f; d[k + 1] = ok ? dv[k / 4].y : 0.0f;
                d[k + 2] = ok ? dv[k / 4].z : 0.0f; d[k + 3] = ok ? dv[k / 4].w : 0.0f;
                b[k] = ok ? bv[k / 4].x : 0.0f; b[k + 1] = ok ? bv[k / 4].y : 0.0f;
                b[k + 2] = ok ? bv[k / 4].z : 0.0f; b[k + 3] = ok ? bv[k / 4].w : 0.0f;
            }
        } else {
            float2 dv[K / 2 + 1], bv[K / 2 + 1];
#pragma unroll
            for (int k = 0; k + 1 < K; k += 2) {
                const int at = min(z + k, nz - 2);
                dv[k / 2] = *(const float2*)(dc + at);
                bv[k / 2] = *(const float2*)(bc + at);
            }
#pragma unroll
            for (int k = 0; k + 1 < K; k += 2) {
                const bool ok = in && z + k < nz;
                d[k] = ok ? dv[k / 2].x : 0.0f; d[k + 1] = ok ? dv[k / 2].y : 0.0f;
                b[k] = ok ? bv[k / 2].x : 0.0f; b[k + 1] = ok ? bv[k / 2].y : 0.0f;
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int at = min(z + k, nz - 1);
        d[k] = dc[at];
        b[k] = bc[at];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bool ok = in && z + k < nz;
        d[k] = ok ? d[k] : 0.0f;
        b[k] = ok ? b[k] : 0.0f;
    }
}

// LDS row of slice z in an array of slices by 16 (columns, parts): 17 doubles each and one
// more every eight slices, so that the lanes of a column, four to eight slices apart, meet
// different banks.
constexpr int slice_row(int z) { return z * 17 + (z >> 3); }

}  // namespace msft
