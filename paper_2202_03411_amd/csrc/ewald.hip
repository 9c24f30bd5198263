// Forward model in spherical coordinates about a detector axis (see ewald.h): the
// column scan with its projection on the z modes, three contractions on the FP64 matrix
// instruction, and the evaluation of each pixel row's Chebyshev series.
//
// The FP64 matrix instruction runs at the FP64 vector rate (78.6 TFLOP/s), one
// 16 x 16 x 4 product in 64 cycles of a SIMD, so its operands can come from the L1 cache
// without staging: one operand of 512 bytes a product.  At the sizes of a pattern
// (128^3 voxels, 512^2 pixels) a whole call is some 0.3 G multiply-adds, and the five
// launches are bound by their own latency and by reading delta and beta once.
#include <hip/hip_runtime.h>

#include "ewald.h"
#include "msft_internal.h"
#include "wave_f64.h"

namespace msft {

namespace {

constexpr int EW_THREADS = 256;
constexpr int EW_WAVES = EW_THREADS / 64;

// The request a workgroup belongs to and its index within it.
__device__ __forceinline__ const EwReq& ew_request(const EwBatch& b, int& item)
{
    int r = 0;
    while (r + 1 < b.n && (int)blockIdx.x >= b.begin[r + 1]) ++r;
    item = (int)blockIdx.x - b.begin[r];
    return b.req[r];
}

// ---------------------------------------------------------------------------
// Scan: w of 16 columns, EW_ZC slices a round, and Z_l = sum_z phi_l(z) exp(-i qc z) w.
//
// Thread (column tid / 16, slices 4 (tid % 16) ..) holds four slices: the 16 lanes of a
// column read 256 contiguous bytes of delta and beta.  The exclusive prefix
// S = sum_{s'<s} (beta + i delta) is the carry of earlier rounds plus a DPP prefix over
// the column's 16 lanes, in FP64; T = exp(-k0 dz S) in FP32 with the phase reduced in
// FP64.  The rotated w goes to LDS (a row of 16 columns per slice, padded to 17 doubles)
// and from there into the matrix instruction: rows are columns, K the slices, columns
// the modes.  Wave w takes Re (w even) or Im of mode tiles w / 2, w / 2 + 2, ...  The
// next round's voxels are loaded before this round's products.
// ---------------------------------------------------------------------------
struct Voxels {
    float d[4], b[4];
};

__device__ __forceinline__ Voxels ew_load(const float* dc, const float* bc, int z, int nz, bool in)
{
    Voxels v;
    if (in && z + 3 < nz && (nz & 3) == 0) {
        const float4 d = *(const float4*)(dc + z), b = *(const float4*)(bc + z);
        v.d[0] = d.x; v.d[1] = d.y; v.d[2] = d.z; v.d[3] = d.w;
        v.b[0] = b.x; v.b[1] = b.y; v.b[2] = b.z; v.b[3] = b.w;
        return v;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool ok = in && z + k < nz;
        v.d[k] = ok ? dc[z + k] : 0.0f;
        v.b[k] = ok ? bc[z + k] : 0.0f;
    }
    return v;
}

constexpr int EW_LD = EW_COLS + 1;

template <int NT>
__global__ __launch_bounds__(EW_THREADS) void ew_scan_kernel(EwBatch batch)
{
    __shared__ double sm[2][EW_ZC * EW_LD];
    int item;
    const EwReq& q = ew_request(batch, item);
    const EwDesc& D = *q.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cl = tid >> 4, zl = (tid & 15) * 4, nz = D.nz;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)item * EW_COLS;
    const bool in = c0 + cl < ncol;
    const int64_t col = in ? c0 + cl : ncol - 1;
    const float* dc = q.delta + col * nz;
    const float* bc = q.beta + col * nz;
    const int ri = wave & 1, t0 = wave >> 1, kzt = D.kzt, strength = D.strength;
    f64x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    double carry_b = 0.0, carry_d = 0.0;
    Voxels v = ew_load(dc, bc, zl, nz, in);
    for (int z0 = 0; z0 < nz; z0 += EW_ZC) {
        double Sb = 0.0, Sd = 0.0;
        if (strength == MSFT_STRENGTH_MSFT) {
            const double sb = ((double)v.b[0] + v.b[1]) + ((double)v.b[2] + v.b[3]);
            const double sd = ((double)v.d[0] + v.d[1]) + ((double)v.d[2] + v.d[3]);
            const double ib = row_prefix_f64(sb), id = row_prefix_f64(sd);
            Sb = carry_b + (ib - sb);
            Sd = carry_d + (id - sd);
            carry_b += row_last_f64(ib);
            carry_d += row_last_f64(id);
        }
        const double2* rot = (const double2*)D.rot + z0 + zl;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float d = v.d[k], b = v.b[k];
            float wr = d, wi = b;
            if (strength != MSFT_STRENGTH_DENSITY) {
                const float chr = d * (d - 2.0f) - b * b, chi = 2.0f * b * (1.0f - d);
                wr = chr;
                wi = chi;
                if (strength == MSFT_STRENGTH_MSFT) {
                    constexpr double kTwoPi = 6.283185307179586476925286766559;
                    const double ph = -D.k0dz64 * Sd;
                    const float mag = expf((float)(-D.k0dz64 * Sb));
                    float sn, cs;
                    sincosf((float)(ph - kTwoPi * rint(ph * (1.0 / kTwoPi))), &sn, &cs);
                    const float tr = mag * cs, ti = mag * sn;
                    wr = chr * tr - chi * ti;
                    wi = chr * ti + chi * tr;
                    Sb += (double)b;
                    Sd += (double)d;
                }
            }
            wr *= D.dV;
            wi *= D.dV;
            const double2 e = rot[k];
            sm[0][(zl + k) * EW_LD + cl] = (double)wr * e.x - (double)wi * e.y;
            sm[1][(zl + k) * EW_LD + cl] = (double)wr * e.y + (double)wi * e.x;
        }
        __syncthreads();
        if (z0 + EW_ZC < nz) v = ew_load(dc, bc, z0 + EW_ZC + zl, nz, in);
        const double* a = sm[ri] + (lane >> 4) * EW_LD + (lane & 15);
        const double* p = D.phiz + (size_t)(z0 + (lane >> 4)) * kzt + t0 * 16 + (lane & 15);
#pragma unroll 4
        for (int kk = 0; kk < EW_ZC / 4; ++kk) {
            const double av = a[4 * kk * EW_LD];
#pragma unroll
            for (int t = 0; t < NT; ++t)
                if ((t0 + 2 * t) * 16 < kzt) acc[t] = mfma_f64(av, p[(size_t)4 * kk * kzt + 32 * t], acc[t]);
        }
        __syncthreads();
    }
    // odd modes carry -i: (re, im) -> (im, -re)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int l = (t0 + 2 * t) * 16 + (lane & 15);
        if (l >= D.kzp) continue;
        const bool odd = l >= D.kze;
        const int comp = odd ? 1 - ri : ri;
        const double sign = odd && ri == 0 ? -1.0 : 1.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t c = c0 + 4 * r + (lane >> 4);
            if (c < ncol) q.ws[c * D.ld + 2 * l + comp] = sign * acc[t][r];
        }
    }
}

// ---------------------------------------------------------------------------
// Modal: Y[N][m][c] = sum_h phi_m(h) (Z[hi] +- Z[lo])[c], c the 2 kzp doubles of a mode
// vector.  A wave takes one N, 16 values of c and two tiles of 16 modes of one parity.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EW_THREADS) void ew_modal_kernel(EwBatch batch)
{
    int item;
    const EwReq& q = ew_request(batch, item);
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, ct = (ld + 15) >> 4, ge = (D.ket + 31) >> 5, go = D.kop ? (D.kot + 31) >> 5 : 0;
    int64_t u = (int64_t)item * EW_WAVES + (threadIdx.x >> 6);
    const int g = (int)(u % (ge + go));
    u /= ge + go;
    const int c = (int)(u % ct) * 16 + li;
    const int N = (int)(u / ct);
    if (N >= D.nN) return;
    const bool odd = g >= ge;
    const int t = (odd ? g - ge : g) * 32, ldt = odd ? D.kot : D.ket;
    const bool two = t + 16 < ldt;
    const double* phi = (odd ? D.phio : D.phie) + t + li;
    const double* z = q.ws + (int64_t)N * D.zsN * ld + min(c, ld - 1);
    const int64_t zs = (int64_t)D.zsM * ld;
    f64x4 a0 = {0.0, 0.0, 0.0, 0.0}, a1 = a0;
    const int last = D.nhM - 1, steps = D.nhMp >> 2;
    for_steps<4>(steps, [&](int ks) {
        const int h = 4 * ks + lk, hc = min(h, last), hi = D.nM - 1 - hc;
        const double vh = z[hi * zs], vl = hi == hc ? 0.0 : z[hc * zs];
        const double b = odd ? vh - vl : vh + vl;
        a0 = mfma_f64(phi[(size_t)h * ldt], b, a0);
        if (two) a1 = mfma_f64(phi[(size_t)h * ldt + 16], b, a1);
    });
    if (c >= ld) return;
    const int kp = odd ? D.kop : D.kep;
    double* y = q.ws + D.offY + ((int64_t)N * D.km + (odd ? D.kep : 0)) * ld + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = t + 4 * r + lk;
        if (m < kp) y[(int64_t)m * ld] = a0[r];
        if (two && m + 16 < kp) y[(int64_t)(m + 16) * ld] = a1[r];
    }
}

// ---------------------------------------------------------------------------
// Nodes: G[a][cos|sin][m][c] = sum_h {cos, sin}(q_N(a) N_h) (Y[hi] +- Y[lo])[m][c].  A
// wave takes 16 of the km * 2 kzp columns and up to two tiles of 16 values of a, both
// parities, so a pair of loads feeds four products.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EW_THREADS) void ew_nodes_kernel(EwBatch batch)
{
    int item;
    const EwReq& q = ew_request(batch, item);
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int ncols = D.km * D.ld, ct = (ncols + 15) >> 4, nap = D.nap, ga = (nap + 31) >> 5;
    const int64_t u = (int64_t)item * EW_WAVES + (threadIdx.x >> 6);
    const int c = (int)(u % ct) * 16 + li, g = (int)(u / ct);
    if (g >= ga) return;
    const bool two = g * 32 + 16 < nap;
    const double* tc = D.cosN + g * 32 + li;
    const double* ts = D.sinN + g * 32 + li;
    const double* y = q.ws + D.offY + min(c, ncols - 1);
    f64x4 e0 = {0.0, 0.0, 0.0, 0.0}, e1 = e0, o0 = e0, o1 = e0;
    const int last = D.nhN - 1, steps = D.nhNp >> 2;
    for_steps<4>(steps, [&](int ks) {
        const int h = 4 * ks + lk, hc = min(h, last), hi = D.nN - 1 - hc;
        const double vh = y[(int64_t)hi * ncols], vl = hi == hc ? 0.0 : y[(int64_t)hc * ncols];
        const double s = vh + vl, d = vh - vl;
        const size_t at = (size_t)h * nap;
        e0 = mfma_f64(tc[at], s, e0);
        o0 = mfma_f64(ts[at], d, o0);
        if (two) {
            e1 = mfma_f64(tc[at + 16], s, e1);
            o1 = mfma_f64(ts[at + 16], d, o1);
        }
    });
    if (c >= ncols) return;
    double* out = q.ws + D.offG + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int a = g * 32 + 4 * r + lk;
        if (a < D.na) {
            out[(int64_t)(2 * a) * ncols] = e0[r];
            out[(int64_t)(2 * a + 1) * ncols] = o0[r];
        }
        if (two && a + 16 < D.na) {
            out[(int64_t)(2 * a + 32) * ncols] = e1[r];
            out[(int64_t)(2 * a + 33) * ncols] = o1[r];
        }
    }
}

// ---------------------------------------------------------------------------
// yz: S[pN][pM](a, b) = sum_l c_l(a, b) sum_{m in pM} c_m(a, b) G[a][pN][m][l].  A wave
// takes one a and 16 values of b (the rows); K runs over the modes m of a parity and
// columns over (l, re | im), both pN sharing the c_m operand; c_l multiplies each
// product tile, the lanes' columns are summed at the end.  The result goes to
// [pixel row][node][4 px + 2 py + (re | im)], px and py the parities along x and y.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EW_THREADS) void ew_yz_kernel(EwBatch batch)
{
    int item;
    const EwReq& q = ew_request(batch, item);
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int bt = D.nbp >> 4, ld = D.ld, nbp = D.nbp, kzp = D.kzp;
    const int64_t u = (int64_t)item * EW_WAVES + (threadIdx.x >> 6);
    const int a = (int)(u / bt), b0 = (int)(u % bt) * 16;
    if (a >= D.na) return;
    const int64_t gs = (int64_t)D.km * ld;
    const double* ga = q.ws + D.offG + 2 * a * gs;
    const double* cz = D.cz + ((size_t)a * nbp + b0 + lk) * kzp;
    double s[2][2][4];   // [pN][pM][row]
#pragma unroll
    for (int k = 0; k < 16; ++k) s[k >> 3][(k >> 2) & 1][k & 3] = 0.0;
#pragma unroll
    for (int pm = 0; pm < 2; ++pm) {
        const int m0 = pm ? D.kep : 0, steps = (pm ? D.kop : D.kep) >> 2;
        const double* cm = D.cm + ((size_t)a * D.km + m0 + lk) * nbp + b0 + li;
        const double* gm = ga + (int64_t)(m0 + lk) * ld;
        for (int c0 = 0; c0 < ld; c0 += 32) {
            const int ca = c0 + li, cb = c0 + 16 + li;
            const int xa = min(ca, ld - 1), xb = min(cb, ld - 1);
            f64x4 ea = {0.0, 0.0, 0.0, 0.0}, eb = ea, oa = ea, ob = ea;
            for_steps<3>(steps, [&](int ks) {
                const double av = cm[(size_t)4 * ks * nbp];
                const double* g = gm + (int64_t)4 * ks * ld;
                ea = mfma_f64(av, g[xa], ea);
                oa = mfma_f64(av, g[gs + xa], oa);
                eb = mfma_f64(av, g[xb], eb);
                ob = mfma_f64(av, g[gs + xb], ob);
            });
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double za = ca < ld ? cz[(size_t)4 * r * kzp + (xa >> 1)] : 0.0;
                const double zb = cb < ld ? cz[(size_t)4 * r * kzp + (xb >> 1)] : 0.0;
                s[0][pm][r] += ea[r] * za + eb[r] * zb;
                s[1][pm][r] += oa[r] * za + ob[r] * zb;
            }
        }
    }
    // sum the lanes of one row with the same re | im (lane bits 1 - 3)
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        double& v = s[k >> 3][(k >> 2) & 1][k & 3];
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 8, 64);
    }
    if (li >= 2) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = b0 + 4 * r + lk;
        if (b >= D.nb) continue;
        const int row = D.uniform ? a : b, node = D.uniform ? b : a;
        double* out = q.ws + D.offA + ((int64_t)row * D.n + node) * 8 + li;
#pragma unroll
        for (int pn = 0; pn < 2; ++pn)
#pragma unroll
            for (int pm = 0; pm < 2; ++pm) out[D.uniform ? 4 * pm + 2 * pn : 4 * pn + 2 * pm] = s[pn][pm][r];
    }
}

// ---------------------------------------------------------------------------
// Eval: one workgroup per pixel row.  Node values -> Chebyshev coefficients (even
// series for px = 0, odd for px = 1) in LDS, then each thread runs the recurrence of
// T_2k and T_2k+1 in x = 2 t^2 - 1 for its column and sums the eight parts:
//   A(sx, sy) = (ee - sx sy oo) - i (sx oe + sy eo)          (px, py)
// for the four mirror pixels.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EW_THREADS) void ew_eval_kernel(EwBatch batch)
{
    extern __shared__ double lds[];   // [2][n][8]: node values, coefficients
    int item;
    const EwReq& q = ew_request(batch, item);
    const EwDesc& D = *q.d;
    const int n = D.n, N = D.det_n, half = D.rows, tid = threadIdx.x;
    const int j = item;
    // rows of this request's pixel range only
    const int jh = N - 1 - j;
    const int64_t lo = (int64_t)j * N, hi = (int64_t)jh * N;
    if ((lo + N <= q.p0 || lo >= q.p1) && (hi + N <= q.p0 || hi >= q.p1)) return;
    double* val = lds;
    double* coef = lds + (size_t)n * 8;
    const double* src = q.ws + D.offA + (int64_t)j * n * 8;
    for (int k = tid; k < n * 8; k += EW_THREADS) val[k] = src[k];
    __syncthreads();
    for (int o = tid; o < n * 8; o += EW_THREADS) {
        const int comp = o & 7, k = o >> 3;
        const double* m = (comp & 4 ? D.dcto : D.dcte) + k;
        double s = 0.0;
#pragma unroll 4
        for (int a = 0; a < n; ++a) s += m[(size_t)a * n] * val[a * 8 + comp];
        coef[o] = s;
    }
    __syncthreads();
    for (int i = tid; i < half; i += EW_THREADS) {
        const double t = D.tq[(int64_t)j * half + i];
        const bool rim = !(t == t);
        const double tt = rim ? 0.0 : t, x2 = 2.0 * (2.0 * tt * tt - 1.0);
        double e0 = 1.0, e1 = 0.5 * x2;           // T_0, T_2
        double o0 = tt, o1 = (x2 - 1.0) * tt;     // T_1, T_3 = (2 x - 1) t
        double s[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) s[c] = 0.0;
#pragma unroll 2
        for (int k = 0; k < n; ++k) {
            const double* C = coef + k * 8;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                s[c] += e0 * C[c];
                s[4 + c] += o0 * C[4 + c];
            }
            const double e2 = x2 * e1 - e0, o2 = x2 * o1 - o0;
            e0 = e1;
            e1 = e2;
            o0 = o1;
            o1 = o2;
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const bool px = !(m & 1), py = !(m & 2);   // the pixel at +u, +v
            const int ii = px ? N - 1 - i : i, jj = py ? jh : j;
            if ((!px && ii == N - 1 - i) || (!py && jj == jh)) continue;   // the middle, done at +
            const double sx = px ? 1.0 : -1.0, sy = py ? 1.0 : -1.0;
            // s: ee re, ee im, eo re, eo im, oe re, oe im, oo re, oo im
            double re = s[0] - sx * sy * s[6] + (sx * s[5] + sy * s[3]);
            double im = s[1] - sx * sy * s[7] - (sx * s[4] + sy * s[2]);
            if (rim) re = im = 0.0;
            const int64_t p = (int64_t)jj * N + ii;
            if (p < q.p0 || p >= q.p1) continue;
            q.intensity[p] = (float)(re * re + im * im);
            if (q.amplitude) ((float2*)q.amplitude)[p] = make_float2((float)re, (float)im);
        }
    }
}

// ---------------------------------------------------------------------------
// Tables of a plan.
// ---------------------------------------------------------------------------

// cos, sin(q_N(a) N_h) [nhNp][nap], zero in the padding.
__global__ void ew_trig_kernel(EwDesc D, const double* ang_a, double k0, double pitch, double* cosN,
                               double* sinN)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int a = (int)(t % D.nap), h = (int)(t / D.nap);
    if (h >= D.nhNp) return;
    double sn = 0.0, cs = 0.0;
    if (a < D.na && h < D.nhN) sincos(k0 * sin(ang_a[a]) * ((D.nN - 1 - 2 * h) * pitch / 2.0), &sn, &cs);
    cosN[t] = cs;
    sinN[t] = sn;
}

struct CoefArgs {
    const double *ang_a, *ang_b, *even, *odd;   // angles; half-axis modes [h][ldE], [h][ldO]
    double* out;                                // out[a * sa + b * sb + m * sm]
    double k0, qc, pitch;
    int na, nb, nbp, n, nh, ke, ko, ldE, ldO, at_odd, zaxis;
    int64_t sa, sb, sm;
};

// Coefficients of exp(-i q r) on an axis's modes: 2 sum_h phi_m(h) cos(q r_h) (even m),
// sin (odd m), the middle voxel of an odd axis once; q = q_M(a, b), or q_z(a, b) - qc.
// Workgroup (16 values of b, one a); the trigonometric values of 64 h at a time in LDS.
__global__ __launch_bounds__(256) void ew_coef_kernel(CoefArgs c)
{
    __shared__ double cs[64][16], sn[64][16];
    const int tid = threadIdx.x, bl = tid & 15, mg = tid >> 4;
    const int a = blockIdx.y, b = blockIdx.x * 16 + bl;
    const double aa = c.ang_a[a], bb = b < c.nb ? c.ang_b[b] : 0.0;
    double q;
    if (c.zaxis) {
        const double sa = sin(0.5 * aa), sb = sin(0.5 * bb);
        q = -2.0 * c.k0 * (sa * sa + cos(aa) * sb * sb) - c.qc;
    } else {
        q = c.k0 * cos(aa) * sin(bb);
    }
    for (int h0 = 0; h0 < c.nh; h0 += 64) {
        const int len = min(64, c.nh - h0);
        for (int h = mg; h < len; h += 16) {
            double s, k;
            sincos(q * ((c.n - 1 - 2 * (h0 + h)) * c.pitch / 2.0), &s, &k);
            const double w = 2 * (h0 + h) + 1 == c.n ? 1.0 : 2.0;
            cs[h][bl] = w * k;
            sn[h][bl] = w * s;
        }
        __syncthreads();
        for (int m = mg; m < c.ke + c.ko; m += 16) {
            const bool odd = m >= c.ke;
            const double* phi = odd ? c.odd + (size_t)h0 * c.ldO + (m - c.ke) : c.even + (size_t)h0 * c.ldE + m;
            const int ldp = odd ? c.ldO : c.ldE;
            double* o = c.out + a * c.sa + b * c.sb + (odd ? c.at_odd + m - c.ke : m) * c.sm;
            double s = h0 ? *o : 0.0;
            for (int h = 0; h < len; ++h) s += phi[(size_t)h * ldp] * (odd ? sn[h][bl] : cs[h][bl]);
            if (b < c.nb) *o = s;
        }
        __syncthreads();
    }
}

int ew_lds(const EwBatch& b, const EwDesc* const* dims)
{
    int n = 0;
    for (int r = 0; r < b.n; ++r) n = dims[r]->n > n ? dims[r]->n : n;
    return n * 16 * (int)sizeof(double);
}

// Workgroups per request by `f`, then one launch over all of them.
template <typename K, typename F>
void ew_launch(K kernel, EwBatch& b, const EwDesc* const* dims, int lds, hipStream_t s, F f)
{
    int64_t total = 0;
    for (int r = 0; r < b.n; ++r) {
        b.begin[r] = (int32_t)total;
        total += f(*dims[r]);
    }
    b.begin[b.n] = (int32_t)total;
    hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(EW_THREADS), lds, s, b);
}

}  // namespace

int launch_ew_scan(EwBatch b, const EwDesc* const* dims, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    int kzt = 0;
    for (int r = 0; r < b.n; ++r) kzt = dims[r]->kzt > kzt ? dims[r]->kzt : kzt;
    auto items = [](const EwDesc& d) { return ceil_div((int64_t)d.nx * d.ny, EW_COLS); };
    const int nt = (kzt / 16 + 1) / 2;   // mode tiles per wave
    if (nt <= 1) ew_launch(ew_scan_kernel<1>, b, dims, 0, s, items);
    else if (nt <= 2) ew_launch(ew_scan_kernel<2>, b, dims, 0, s, items);
    else if (nt <= 4) ew_launch(ew_scan_kernel<4>, b, dims, 0, s, items);
    else ew_launch(ew_scan_kernel<EW_MAX_KZ / 32>, b, dims, 0, s, items);
    return (int)hipGetLastError();
}

int launch_ew_contract(EwBatch b, const EwDesc* const* dims, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    ew_launch(ew_modal_kernel, b, dims, 0, s, [](const EwDesc& d) {
        const int64_t g = ceil_div(d.ket, 32) + (d.kop ? ceil_div(d.kot, 32) : 0);
        return ceil_div(g * ceil_div(d.ld, 16) * d.nN, EW_WAVES);
    });
    ew_launch(ew_nodes_kernel, b, dims, 0, s, [](const EwDesc& d) {
        return ceil_div(ceil_div((int64_t)d.km * d.ld, 16) * ceil_div(d.nap, 32), EW_WAVES);
    });
    ew_launch(ew_yz_kernel, b, dims, 0, s,
              [](const EwDesc& d) { return ceil_div((int64_t)d.na * (d.nbp / 16), EW_WAVES); });
    ew_launch(ew_eval_kernel, b, dims, ew_lds(b, dims), s, [](const EwDesc& d) { return (int64_t)d.rows; });
    return (int)hipGetLastError();
}

int launch_ew_tables(const EwHost& h, const EwDesc& D, const EwTables& t, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(ew_trig_kernel, dim3((unsigned)ceil_div((int64_t)D.nhNp * D.nap, 256)), dim3(256), 0, s,
                       D, t.ang_a, h.k0, h.pitchN, t.cosN, t.sinN);
    const dim3 grid((unsigned)(D.nbp / 16), (unsigned)D.na);
    CoefArgs c;
    c.ang_a = t.ang_a;
    c.ang_b = t.ang_b;
    c.k0 = h.k0;
    c.qc = h.qc;
    c.na = D.na;
    c.nb = D.nb;
    c.nbp = D.nbp;
    c.even = D.phie;
    c.odd = D.phio;
    c.ldE = D.ket;
    c.ldO = D.kot;
    c.out = t.cm;
    c.pitch = h.pitchM;
    c.n = D.nM;
    c.nh = D.nhM;
    c.ke = D.kep;
    c.ko = D.kop;
    c.at_odd = D.kep;
    c.zaxis = 0;
    c.sa = (int64_t)D.km * D.nbp;
    c.sb = 1;
    c.sm = D.nbp;
    hipLaunchKernelGGL(ew_coef_kernel, grid, dim3(256), 0, s, c);
    c.even = t.phize;
    c.odd = t.phizo;
    c.ldE = D.kze;
    c.ldO = D.kz - D.kze;
    c.out = t.cz;
    c.pitch = h.pitchZ;
    c.n = D.nz;
    c.nh = (D.nz + 1) / 2;
    c.ke = D.kze;
    c.ko = D.kz - D.kze;
    c.at_odd = D.kze;
    c.zaxis = 1;
    c.sa = (int64_t)D.nbp * D.kzp;
    c.sb = D.kzp;
    c.sm = 1;
    hipLaunchKernelGGL(ew_coef_kernel, grid, dim3(256), 0, s, c);
    return (int)hipGetLastError();
}

}  // namespace msft
