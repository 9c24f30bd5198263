// gfx950 shape renderers (Sec. 5.2): the sample's delta, beta on the centred voxel
// grid, ahead of the column scan, and the gradient of a loss with respect to the
// star body's harmonic coefficients.
//
//  render_sh_kernel        r_s(theta, phi) = r0 (1 + sum c_lm Y_lm), occupancy, delta/beta
//  render_sh_grad_kernel   per-workgroup partial sums of dL/dc_lm (FP64 partials)
//  render_sh_grad_reduce   the partials summed in a fixed order
//  render_ellipsoid_kernel quadric body, hard or soft
//  render_volume_kernel    a voxel map on its own grid, resampled (trilinear)
//
// The star body's kernels take eight mirror voxels to a thread, the others one voxel;
// directions, radii and the harmonic sums in FP64, outputs in FP32.
#include <hip/hip_runtime.h>

#include "msft_internal.h"
#include "wave_f64.h"

namespace msft {

// Voxel v = (a * ny + b) * nz + k -> centre, distance, cos(theta), cos/sin(phi);
// the origin looks along +z.
struct VoxelDir {
    double x, y, z, r, ct, st, cp, sp;
};

__device__ __forceinline__ VoxelDir voxel_dir(const RenderGrid& g, int64_t v)
{
    const int k = (int)(v % g.nz);
    const int64_t ab = v / g.nz;
    const int b = (int)(ab % g.ny), a = (int)(ab / g.ny);
    const double x = ((double)(2 * a + 1 - g.nx) * g.dx) / 2.0;
    const double y = ((double)(2 * b + 1 - g.ny) * g.dy) / 2.0;
    const double z = ((double)(2 * k + 1 - g.nz) * g.dz) / 2.0;
    VoxelDir d;
    d.x = x;
    d.y = y;
    d.z = z;
    const double rxy = sqrt(x * x + y * y);
    d.r = sqrt(x * x + y * y + z * z);
    if (d.r > 0.0) {
        d.ct = z / d.r;
        d.st = rxy / d.r;
    } else {
        d.ct = 1.0;
        d.st = 0.0;
    }
    if (rxy > 0.0) {
        d.cp = x / rxy;
        d.sp = y / rxy;
    } else {
        d.cp = 1.0;
        d.sp = 0.0;
    }
    return d;
}

__device__ __forceinline__ double occupancy(double rs, double r, double edge)
{
    if (edge <= 0.0) return r <= rs ? 1.0 : 0.0;
    return 1.0 / (1.0 + exp(-(rs - r) / edge));
}

// ---------------------------------------------------------------------------
// The star body.  The voxels (+-x, +-y, +-z) share r, the powers of sin and cos(theta) and
// cos and sin(m phi) up to signs, so a thread takes the eight of one octant: it sums
// the harmonics by their parities (z: l - m, x: m or m + 1, y: cos or sin) and the eight
// radii are the parities' signed sums.  Y_lm = norm sin^m p_lm {cos, sin}(m phi) with
// monic p: p_l = cos p_{l-1} - ((l-1)^2 - m^2) / (4 (l-1)^2 - 1) p_{l-2}, two operations.
// Bound by FP64 operations, about 90 a voxel with the exponential (one voxel to a thread
// took some 570): 128^3, l <= 8, forward 57 -> 12.7 us, gradient 138 -> 19.0 us.
// ---------------------------------------------------------------------------
constexpr int SH_GRAD_RESIDENT = 256;
constexpr int sh_at(int L, int l, int m) { return m * (L + 1) - m * (m - 1) / 2 + l - m; }
constexpr int sh_pairs(int L) { return (L + 1) * (L + 2) / 2; }
constexpr double sh_gamma(int l, int m)
{
    return ((double)(l - 1) * (l - 1) - (double)m * m) / (4.0 * (l - 1) * (l - 1) - 1.0);
}

// exp(x), |x| <= 700: range reduction and the Taylor series on |r| <= ln(2) / 2 to
// r^13 / 13! (remainder 4e-18).
__device__ __forceinline__ double exp_f64(double x)
{
    const double n = rint(x * 1.4426950408889634074);
    double r = __builtin_fma(n, -0.69314718055994528623, x);
    r = __builtin_fma(n, -2.3190468138462996e-17, r);
    double p = 1.0 / 6227020800.0;
    p = __builtin_fma(p, r, 1.0 / 479001600.0);
    p = __builtin_fma(p, r, 1.0 / 39916800.0);
    p = __builtin_fma(p, r, 1.0 / 3628800.0);
    p = __builtin_fma(p, r, 1.0 / 362880.0);
    p = __builtin_fma(p, r, 1.0 / 40320.0);
    p = __builtin_fma(p, r, 1.0 / 5040.0);
    p = __builtin_fma(p, r, 1.0 / 720.0);
    p = __builtin_fma(p, r, 1.0 / 120.0);
    p = __builtin_fma(p, r, 1.0 / 24.0);
    p = __builtin_fma(p, r, 1.0 / 6.0);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    p = __builtin_fma(p, r, 1.0);
    return __builtin_ldexp(p, (int)n);
}

__device__ __forceinline__ double reciprocal(double d)
{
    double y = __builtin_amdgcn_rcp(d);
    y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
}

// Item t of plane `ha`: the octant's voxel at the non-negative coordinates and its seven
// mirrors, v[4 kz + 2 kx + ky] (k = 1: the mirrored side).  An axis's middle voxel is its
// own mirror: `own` says which of the eight are there once.
struct Octant {
    double r, ct, px, py;   // distance; z, x and y over it (+z at the origin)
    int64_t v[8];
    bool in, two[3];        // within the plane; z, x, y have a mirror of their own

    __device__ __forceinline__ void at(const RenderGrid& g, int ha, uint32_t t)
    {
        const uint32_t nyh = (uint32_t)(g.ny + 1) >> 1, nzh = (uint32_t)(g.nz + 1) >> 1;
        in = t < nyh * nzh;
        if (!in) t = nyh * nzh - 1;
        const int hb = (int)(t / nzh), hk = (int)(t - (uint32_t)hb * nzh);
        const int a = g.nx - 1 - ha, b = g.ny - 1 - hb, k = g.nz - 1 - hk;
        two[0] = k != hk;
        two[1] = a != ha;
        two[2] = b != hb;
        const double x = ((double)(2 * a + 1 - g.nx) * g.dx) / 2.0;
        const double y = ((double)(2 * b + 1 - g.ny) * g.dy) / 2.0;
        const double z = ((double)(2 * k + 1 - g.nz) * g.dz) / 2.0;
        r = sqrt(x * x + y * y + z * z);
        const double i = r > 0.0 ? reciprocal(r) : 0.0;
        ct = r > 0.0 ? z * i : 1.0;
        px = x * i;
        py = y * i;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = ((int64_t)(e & 2 ? ha : a) * g.ny + (e & 1 ? hb : b)) * g.nz + (e & 4 ? hk : k);
    }
    __device__ __forceinline__ bool own(int e) const
    {
        return in && (!(e & 4) || two[0]) && (!(e & 2) || two[1]) && (!(e & 1) || two[2]);
    }
};

// Sums and differences over the three parities: w[4 z + 2 x + y].
__device__ __forceinline__ void octant_signs(double* w)
{
#pragma unroll
    for (int s = 1; s < 8; s *= 2)
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (!(e & s)) {
                const double a = w[e], b = w[e | s];
                w[e] = a + b;
                w[e | s] = a - b;
            }
}

// norm times coefficient of (l, m) and (l, -m) at 2 sh_at(L, l, m), zero beyond lmax.
template <int L>
__device__ __forceinline__ void sh_coefficients(const ShArgs& s, const float* coeffs, double* c)
{
    for (int k = threadIdx.x; k < 2 * sh_pairs(L); k += blockDim.x) {
        int m = 0, i = k >> 1;
        while (i > L - m) i -= L + 1 - m++;
        const int l = m + i;
        double v = 0.0;
        if (l <= s.lmax && (m > 0 || !(k & 1))) v = s.norm[l * SH_TABLE + m] * (double)coeffs[l * l + l + (k & 1 ? -m : m)];
        c[k] = v;
    }
}

// 1 + sum c_lm Y_lm at an octant's eight voxels.
template <int L>
__device__ __forceinline__ void sh_radii(const Octant& o, const double* c, double* R)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) R[e] = 0.0;
    double cm = 1.0, sm = 0.0;   // sin^m(theta) {cos, sin}(m phi)
#pragma unroll
    for (int m = 0; m <= L; ++m) {
        if (m > 0) {
            const double c2 = cm * o.px - sm * o.py;
            sm = sm * o.px + cm * o.py;
            cm = c2;
        }
        
        double u[2] = {0.0, 0.0}, v[2] = {0.0, 0.0}, p2 = 0.0, p1 = 0.0;
#pragma unroll
        for (int l = m; l <= L; ++l) {
            const double p = l == m ? 1.0 : l == m + 1 ? o.ct : __builtin_fma(o.ct, p1, -sh_gamma(l, m) * p2);
            p2 = p1;
            p1 = p;
            const double* k = c + 2 * sh_at(L, l, m);
            u[(l - m) & 1] += k[0] * p;
            if (m > 0) v[(l - m) & 1] += k[1] * p;
        }
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            if (z > L - m) continue;
            R[4 * z + 2 * (m & 1)] += cm * u[z];
            if (m > 0) R[4 * z + 2 * (~m & 1) + 1] += sm * v[z];
        }
    }
    R[0] += 1.0;
    octant_signs(R);
}

// exp(-x) of the soft occupancy 1 / (1 + exp(-x)), x = (rs - r) / edge held to +-700 (NaN
// passes).
__device__ __forceinline__ double edge_exp(double rs, double r, double inv_edge)
{
    double x = (r - rs) * inv_edge;
    x = x > 700.0 ? 700.0 : x;
    return exp_f64(x < -700.0 ? -700.0 : x);
}

template <int L>
__global__ __launch_bounds__(256) void render_sh_kernel(ShArgs s, const float* coeffs, float* delta,
                                                        float* beta)
{
    __shared__ double c[2 * sh_pairs(L)];
    sh_coefficients<L>(s, coeffs, c);
    __syncthreads();
    Octant o;
    o.at(s.g, blockIdx.y, blockIdx.x * 256 + threadIdx.x);
    double R[8];
    sh_radii<L>(o, c, R);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const double rs = s.r0 * R[e];
        double occ;
        if (s.inv_edge > 0.0) occ = reciprocal(1.0 + edge_exp(rs, o.r, s.inv_edge));
        else occ = o.r <= rs ? 1.0 : 0.0;
        if (!o.own(e)) continue;
        delta[o.v[e]] = (float)(s.g.delta0 * occ);
        beta[o.v[e]] = (float)(s.g.beta0 * occ);
    }
}

// a, b -> a's sums of the two halves of a wave in the lower half, b's in the upper
// (HALF = 32); the same of neighbouring rows of 16 lanes (HALF = 16).
template <int HALF>
__device__ __forceinline__ double swap_add(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    auto lo = HALF == 32 ? __builtin_amdgcn_permlane32_swap((unsigned)ua, (unsigned)ub, false, false)
                         : __builtin_amdgcn_permlane16_swap((unsigned)ua, (unsigned)ub, false, false);
    auto hi = HALF == 32 ? __builtin_amdgcn_permlane32_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false)
                         : __builtin_amdgcn_permlane16_swap((unsigned)(ua >> 32), (unsigned)(ub >> 32), false, false);
    return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
}

__device__ __forceinline__ double row_sum_f64(double v)
{
    v += dpp_f64<0x128, 0xF>(v);   // row_ror 8, 4, 2, 1
    v += dpp_f64<0x124, 0xF>(v);
    v += dpp_f64<0x122, 0xF>(v);
    return v + dpp_f64<0x121, 0xF>(v);
}

// dL/dc_lm = sum_v (gd delta0 + gb beta0) o (1 - o) / edge r0 Y_lm for M0 <= m < M1.  A
// thread walks octants in a grid stride: the eight weights' parity sums times p_lm, in FP64
// registers, summed over the wave by halves, quarters and rows, over the workgroup's waves
// in LDS, into partials [block][coeff].  m is cut in two for L = 12, whose 169 sums do not
// fit the registers.
template <int L, int M0, int M1>
__global__ __launch_bounds__(256, 1) void render_sh_grad_kernel(ShArgs s, const float* coeffs,
                                                                const float* gd, const float* gb,
                                                                double* partial)
{
    constexpr int FIRST = sh_at(L, M0, M0), COUNT = 2 * (sh_at(L, M1, M1) - FIRST);
    constexpr int S1 = (COUNT + 1) / 2, S2 = (S1 + 1) / 2;
    __shared__ double c[2 * sh_pairs(L)];
    __shared__ double wsum[4][4 * S2];
    sh_coefficients<L>(s, coeffs, c);
    __syncthreads();
    double acc[4 * S2];
#pragma unroll
    for (int k = 0; k < 4 * S2; ++k) acc[k] = 0.0;
    const uint32_t plane = ((uint32_t)(s.g.ny + 1) >> 1) * ((uint32_t)(s.g.nz + 1) >> 1);
    const uint32_t chunks = (plane + 255) / 256, total = chunks * ((uint32_t)(s.g.nx + 1) >> 1);
    const double scale = s.inv_edge * s.r0;
    for (uint32_t k = blockIdx.x; k < total; k += gridDim.x) {
        const uint32_t ha = k / chunks;
        Octant o;
        o.at(s.g, (int)ha, (k - ha * chunks) * 256 + threadIdx.x);
        float d[8], b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            d[e] = gd[o.v[e]];
            b[e] = gb[o.v[e]];
        }
        // an offset the compiler cannot see through: the coefficients, the same each time,
        // would be kept in registers (2 (L + 1)^2 of them)
        int opaque = 0;
        asm volatile("" : "+v"(opaque));
        double w[8];
        sh_radii<L>(o, c + opaque, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const double x = edge_exp(s.r0 * w[e], o.r, s.inv_edge), occ = reciprocal(1.0 + x);
            const double g = (double)d[e] * s.g.delta0 + (double)b[e] * s.g.beta0;
            w[e] = o.own(e) ? g * (x * occ) * occ * scale : 0.0;   // 1 - o = exp(-x) o
        }
        octant_signs(w);
        double cm = 1.0, sm = 0.0;
#pragma unroll
        for (int m = 0; m < M1; ++m) {
            if (m > 0) {
                const double c2 = cm * o.px - sm * o.py;
                sm = sm * o.px + cm * o.py;
                cm = c2;
            }
            if (m < M0) continue;
            __builtin_amdgcn_sched_barrier(0);
            double u[2], v[2], p2 = 0.0, p1 = 0.0;
#pragma unroll
            for (int z = 0; z < 2; ++z) {
                u[z] = cm * w[4 * z + 2 * (m & 1)];
                v[z] = sm * w[4 * z + 2 * (~m & 1) + 1];
            }
#pragma unroll
            for (int l = m; l <= L; ++l) {
                const double p = l == m ? 1.0 : l == m + 1 ? o.ct : __builtin_fma(o.ct, p1, -sh_gamma(l, m) * p2);
                p2 = p1;
                p1 = p;
                const int at = 2 * (sh_at(L, l, m) - FIRST);
                acc[at] += p * u[(l - m) & 1];
                if (m > 0) acc[at + 1] += p * v[(l - m) & 1];
            }
        }
    }
    // value 4 j + i of the wave ends in row 2 (i & 1) + (i >> 1) of register j
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < S2; ++j) {
        const double v = row_sum_f64(swap_add<16>(swap_add<32>(acc[4 * j], acc[4 * j + 1]),
                                                  swap_add<32>(acc[4 * j + 2], acc[4 * j + 3])));
        const int row = lane >> 4;
        if ((lane & 15) == 0) wsum[wave][4 * j + (row >> 1) + 2 * (row & 1)] = v;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < COUNT; k += 256) {
        int m = M0, i = k >> 1;
        while (i > L - m) i -= L + 1 - m++;
        const int l = m + i;
        if (m == 0 && (k & 1)) continue;
        partial[(int64_t)blockIdx.x * MAX_SH_COEFFS + l * l + l + (k & 1 ? -m : m)] =
            s.norm[l * SH_TABLE + m] * (((wsum[0][k] + wsum[1][k]) + wsum[2][k]) + wsum[3][k]);
    }
}

// One workgroup per coefficient: thread t adds the partials b = t, t + 256, ... in
// FP64, then a fixed pairwise tree over the 256 threads.  The order is fixed, so
// repeated calls give the same bits.  (One thread per coefficient walking all the
// partials waited on one load at a time: most of the gradient's time.)
__global__ __launch_bounds__(256) void render_sh_grad_reduce(const double* partial, int nblocks, float* grad)
{
    __shared__ double red[256];
    const int k = blockIdx.x, t = threadIdx.x;
    double s = 0.0;
    for (int b = t; b < nblocks; b += 256) s += partial[(int64_t)b * MAX_SH_COEFFS + k];
    red[t] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h) red[t] += red[t + h];
        __syncthreads();
    }
    if (t == 0) grad[k] = (float)red[0];
}

__global__ __launch_bounds__(256) void render_ellipsoid_kernel(EllArgs e, float* delta, float* beta)
{
    const int64_t nv = (int64_t)e.g.nx * e.g.ny * e.g.nz;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const VoxelDir d = voxel_dir(e.g, v);
    // the voxel centre and its unit direction (+z at the origin) in body coordinates
    const double ux = d.st * d.cp, uy = d.st * d.sp, uz = d.ct;
    double rho2 = 0.0, e2 = 0.0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const double pj = d.x * e.rot[0 * 3 + j] + d.y * e.rot[1 * 3 + j] + d.z * e.rot[2 * 3 + j];
        rho2 += (pj / e.ax[j]) * (pj / e.ax[j]);
        const double uj = ux * e.rot[0 * 3 + j] + uy * e.rot[1 * 3 + j] + uz * e.rot[2 * 3 + j];
        e2 += (uj / e.ax[j]) * (uj / e.ax[j]);
    }
    double o;
    if (e.g.edge <= 0.0) o = rho2 <= 1.0 ? 1.0 : 0.0;
    else o = occupancy(1.0 / sqrt(e2), d.r, e.g.edge);
    delta[v] = (float)(e.g.delta0 * o);
    beta[v] = (float)(e.g.beta0 * o);
}

// Volume map: trilinear interpolation between the centres of a source grid
// (also centred on the origin), zero beyond it; FP64 coordinates and weights.
__global__ __launch_bounds__(256) void render_volume_kernel(VolArgs a, const float* sd,
                                                            const float* sb, float* delta, float* beta)
{
    const int64_t nv = (int64_t)a.g.nx * a.g.ny * a.g.nz;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    const VoxelDir d = voxel_dir(a.g, v);
    const double fx = d.x / a.sdx + (a.sx - 1) / 2.0;
    const double fy = d.y / a.sdy + (a.sy - 1) / 2.0;
    const double fz = d.z / a.sdz + (a.sz - 1) / 2.0;
    const double ax = floor(fx), ay = floor(fy), az = floor(fz);
    const double wx = fx - ax, wy = fy - ay, wz = fz - az;
    double vd = 0.0, vb = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int64_t x = (int64_t)ax + i, y = (int64_t)ay + j, z = (int64_t)az + k;
                if (x < 0 || x >= a.sx || y < 0 || y >= a.sy || z < 0 || z >= a.sz) continue;
                const double w = (i ? wx : 1.0 - wx) * (j ? wy : 1.0 - wy) * (k ? wz : 1.0 - wz);
                const int64_t s = (x * a.sy + y) * a.sz + z;
                vd += w * (double)sd[s];
                vb += w * (double)sb[s];
            }
    delta[v] = (float)vd;
    beta[v] = (float)vb;
}

int launch_render_volume(const VolArgs& a, const float* sd, const float* sb, float* delta,
                         float* beta, void* stream)
{
    const int64_t nv = (int64_t)a.g.nx * a.g.ny * a.g.nz;
    hipLaunchKernelGGL(render_volume_kernel, dim3((unsigned)ceil_div(nv, 256)), dim3(256), 0,
                       (hipStream_t)stream, a, sd, sb, delta, beta);
    return (int)hipGetLastError();
}

int launch_render_sh(const ShArgs& s, const float* coeffs, float* delta, float* beta, void* stream)
{
    const dim3 grid((unsigned)ceil_div((int64_t)((s.g.ny + 1) / 2) * ((s.g.nz + 1) / 2), 256), (unsigned)((s.g.nx + 1) / 2));
    hipStream_t st = (hipStream_t)stream;
    if (s.lmax <= 8)
        hipLaunchKernelGGL(render_sh_kernel<8>, grid, dim3(256), 0, st, s, coeffs, delta, beta);
    else
        hipLaunchKernelGGL(render_sh_kernel<MAX_SH_L>, grid, dim3(256), 0, st, s, coeffs, delta, beta);
    return (int)hipGetLastError();
}

int launch_render_sh_grad(const ShArgs& s, const float* coeffs, const float* gd, const float* gb,
                          float* grad, double* partial, int nblocks, void* stream)
{
    hipStream_t st = (hipStream_t)stream;
    // the sums take over 256 registers a lane, so one workgroup fits a CU: one for each (the
    // 128^3 gradient takes 19.0 us, with two for each 22.6)
    nblocks = nblocks < SH_GRAD_RESIDENT ? nblocks : SH_GRAD_RESIDENT;
    const dim3 grid((unsigned)nblocks);
    if (s.lmax <= 8) {
        hipLaunchKernelGGL((render_sh_grad_kernel<8, 0, 9>), grid, dim3(256), 0, st, s, coeffs, gd, gb, partial);
    } else {
        constexpr int CUT = 4;   // 92 sums below m = 4, 90 from there on
        hipLaunchKernelGGL((render_sh_grad_kernel<MAX_SH_L, 0, CUT>), grid, dim3(256), 0, st, s, coeffs, gd, gb, partial);
        hipLaunchKernelGGL((render_sh_grad_kernel<MAX_SH_L, CUT, SH_TABLE>), grid, dim3(256), 0, st, s, coeffs, gd, gb,
                           partial);
    }
    const int nc = (s.lmax + 1) * (s.lmax + 1);
    hipLaunchKernelGGL(render_sh_grad_reduce, dim3((unsigned)nc), dim3(256), 0, st, (const double*)partial,
                       nblocks, grad);
    return (int)hipGetLastError();
}

int launch_render_ellipsoid(const EllArgs& e, float* delta, float* beta, void* stream)
{
    const int64_t nv = (int64_t)e.g.nx * e.g.ny * e.g.nz;
    hipLaunchKernelGGL(render_ellipsoid_kernel, dim3((unsigned)ceil_div(nv, 256)), dim3(256), 0,
                       (hipStream_t)stream, e, delta, beta);
    return (int)hipGetLastError();
}

}  // namespace msft
