// Adjoint of the spherical-coordinate forward model (see ewald.h): the stages of the
// forward transposed, in FP64, and the column walk of the chain rule.
//
//   rows   C(row, k)  = sum over the row's pixels of T_k(t) h
//          (h = g conj(A), folded over the four mirror pixels)
//   coef   S(r, a)    = sum_k D[a][k] sum over the rows of W[row][r] C
//   yz     G_ml(a)    = sum_b c_m(a, b) c_l(a, b) S(a, b)
//   nodes  Y_ml(N)    = sum_a {cos, sin}(q_N(a) N) G_ml(a)
//   modal  Z_l(N, M)  = sum_m phi_m(M) Y_ml(N)
//   walk   R(z)       = exp(-i qc z) sum_l phi_l(z) Z_l, then along each column
//          dL/d delta, dL/d beta from R (Eqs. (7)-(9))
//
// Every array takes the place of the forward's of the same letter (C its parts in planes).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "ewald.h"
#include "msft_internal.h"
#include "wave_f64.h"

namespace msft {

namespace {

constexpr int EA_THREADS = 256;
constexpr int EA_WAVES = EA_THREADS / 64;

// ---------------------------------------------------------------------------
// Rows: one workgroup per pixel row, 256 columns at a time, 64 to a wave.  A lane folds h
// of its column's mirror pixels into the eight parts and runs the recurrences of T_2k and
// T_2k+1, eight orders at a time into the wave's own LDS (a row of pixels per order: the
// writes are contiguous, the reads of 16 orders by 4 pixels meet distinct banks).  The
// sums over pixels are products on the four-block matrix instruction, blocks 0 and 1 the
// even orders, 2 and 3 the odd ones with their four parts: no lane is idle, where on the
// 16 x 16 one three quarters of the columns would be.  The waves' sums of 32 orders meet
// in LDS.
// ---------------------------------------------------------------------------
constexpr int RW_ORDERS = 32;

__global__ __launch_bounds__(EA_THREADS) void ew_rows_kernel(EwAdj q)
{
    __shared__ double T[EA_WAVES][16][65], Hs[EA_WAVES][8][65], sums[EA_WAVES][RW_ORDERS * 8];
    const EwDesc& D = *q.d;
    const int n = D.n, N = D.det_n, half = D.rows, tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int j = blockIdx.x, jh = N - 1 - j, li = lane & 15, lk = lane >> 4, par = li >> 3, lc = lane & 3;
    const gcdouble tq = as_global(D.tq) + (int64_t)j * half;
    const float __attribute__((address_space(1)))* g = as_global(q.grad_intensity);
    const float __attribute__((address_space(1)))* A = as_global(q.amplitude);
    gdouble C = as_global(q.ws) + D.offC + ((int64_t)(tid & 7) * half + j) * n + (tid >> 3);   // [part][row][order]
    for (int i0 = 0; i0 < half; i0 += EA_THREADS) {
        const int i = i0 + tid;
        const double t = tq[min(i, half - 1)];
        const bool rim = !(t == t) || i >= half;
        double H[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) H[c] = 0.0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const bool px = !(m & 1), py = !(m & 2);   // the pixel at +u, +v
            const int ii = px ? N - 1 - i : i;
            if (rim || (!px && ii == N - 1 - i) || (!py && j == jh)) continue;
            const double sx = px ? 1.0 : -1.0, sy = py ? 1.0 : -1.0;
            const int64_t p = (int64_t)(py ? jh : j) * N + ii;
            const double gv = g[p], hr = gv * (double)A[2 * p], hi = -gv * (double)A[2 * p + 1];
            // transposes of ee - sx sy oo - i (sx oe + sy eo)
            H[0] += hr;
            H[1] += hi;
            H[2] += sy * hi;
            H[3] -= sy * hr;
            H[4] += sx * hi;
            H[5] -= sx * hr;
            H[6] -= sx * sy * hr;
            H[7] -= sx * sy * hi;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) Hs[wave][c][lane] = H[c];
        const double tt = rim ? 0.0 : t, x2 = 2.0 * (2.0 * tt * tt - 1.0);
        double e0 = 1.0, e1 = 0.5 * x2, o0 = tt, o1 = (x2 - 1.0) * tt;
        for (int k0 = 0; k0 < n; k0 += RW_ORDERS) {
#pragma unroll 1
            for (int kb = 0; kb < RW_ORDERS; kb += 8) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    T[wave][k][lane] = e0;
                    T[wave][8 + k][lane] = o0;
                    const double e2 = x2 * e1 - e0, o2 = x2 * o1 - o0;
                    e0 = e1;
                    e1 = e2;
                    o0 = o1;
                    o1 = o2;
                }
                __builtin_amdgcn_wave_barrier();   // the wave's own LDS, in order
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 16; ++s)
                    acc[s & 3] = mfma_f64_4b(T[wave][li][4 * s + lk], Hs[wave][4 * par + lc][4 * s + lk], acc[s & 3]);
                __builtin_amdgcn_wave_barrier();
                sums[wave][(kb + (li & 4) + lk) * 8 + 4 * par + lc] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
            __syncthreads();
            const double s = (sums[0][tid] + sums[1][tid]) + (sums[2][tid] + sums[3][tid]);
            if (k0 + (tid >> 3) < n) C[k0] = i0 ? C[k0] + s : s;
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// Coef transposed: S[comp][r][a] = sum_k D[a][k] sum over rows of W[row][r] C[comp][row][k]
// for 16 row nodes and one part: 16 waves, four to the rows and four to the tiles of 16
// orders k, their sums through LDS (a row of 16 row nodes per order, padded to 17), then a
// wave to each tile of 16 nodes a.
// ---------------------------------------------------------------------------
constexpr int CA_THREADS = 1024;
constexpr int CA_RED = 3 * 4 * 4 * 64;   // rows' part, tile, its values
static_assert((EW_MAX_NODES * 17 + CA_RED) * sizeof(double) <= EW_LDS, "one workgroup's LDS at the most nodes");

__global__ __launch_bounds__(CA_THREADS) void ew_coef_adj_kernel(EwAdj q)
{
    extern __shared__ double lds[];              // [n][17]
    __shared__ double red[3][4][4 * 64];
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int n = D.n, nr = D.nr, rowsp = D.rowsp, np = (n + 15) & ~15;
    const int comp = blockIdx.x & 7, r0 = (blockIdx.x >> 3) * 16, part = wave >> 2;
    const int px = comp >> 2, py = (comp >> 1) & 1, last = D.rows - 1;
    const gcdouble w = as_global(py ? D.wro : D.wre) + (int64_t)r0 * rowsp;
    const gcdouble C = as_global(q.ws) + D.offC + (int64_t)comp * D.rows * n;
    const uint32_t ow = 8 * (li * rowsp + lk);
    const int steps = rowsp >> 4;   // of four rows, per part
    for (int t0 = 0; t0 < np; t0 += 64) {
        const int k = min(t0 + 16 * (wave & 3) + li, n - 1);
        f64x4 t = F64X4_ZERO;
        for_steps<8>(steps, [&](int ks) {
            const int j = 4 * (part * steps + ks);   // W is zero for rows past the last
            t = mfma_f64(load_at(w + j, ow), C[min(j + lk, last) * n + k], t);
        });
        if (part)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[part - 1][wave & 3][r * 64 + lane] = t[r];
        __syncthreads();
        if (!part && t0 + 16 * wave + li < n)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                lds[(t0 + 16 * wave + li) * 17 + 4 * r + lk] =
                    ((t[r] + red[0][wave][r * 64 + lane]) + red[1][wave][r * 64 + lane]) + red[2][wave][r * 64 + lane];
        __syncthreads();
    }
    const gcdouble m = as_global(px ? D.dcto : D.dcte);
    gdouble out = as_global(q.ws) + D.offS + (int64_t)comp * nr * n;
    for (int a0 = 16 * wave; a0 < n; a0 += 16 * (CA_THREADS / 64)) {
        f64x4 t = F64X4_ZERO;
        for_steps<8>((n + 3) >> 2, [&](int ks) {   // D is zero for k >= n
            const int k = 4 * ks;
            t = mfma_f64(lds[min(k + lk, n - 1) * 17 + li], load_at(m + (int64_t)a0 * np + k, 8 * (li * np + lk)), t);
        });
        if (a0 + li < n)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r0 + 4 * r + lk < nr) out[(int64_t)(r0 + 4 * r + lk) * n + a0 + li] = t[r];
    }
}

// ---------------------------------------------------------------------------
// yz transposed: G[a][pN][m][(l, ri)] = sum_b c_m(a, b) c_l(a, b) S(a, b)[pN][pM(m)][ri].
// A workgroup takes one a, one pN and two tiles of 16 columns (l, ri); a wave one parity
// of m and one tile of 16 of its modes; K runs over b, the second operand formed from
// c_l and S.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_yz_adj_kernel(EwAdj q)
{
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, cg = (ld + 31) >> 5, mg = (max(D.kep, D.kop) + 31) >> 5;
    // the workgroups of one a follow each other on one XCD
    int u = blockIdx.x >> 3;
    const int g = u % cg;
    u /= cg;
    const int pm = wave & 1, m0 = u % mg * 32 + 16 * (wave >> 1), kp = pm ? D.kop : D.kep;
    u /= mg;
    const int pn = u & 1, a = (u >> 1) * 8 + (blockIdx.x & 7);
    if (a >= D.na || m0 >= kp) return;   // nothing waits for a wave that is done
    const int nbp = D.nbp, kzp = D.kzp, nb = D.nb, uni = D.uniform;
    // rows past the parity's modes read its last and are not stored
    const gcdouble cm = as_global(D.cm) + ((int64_t)a * D.km + (pm ? D.kep : 0) + m0) * nbp;
    const uint32_t om = 8 * (min(li, kp - 1 - m0) * nbp + lk);
    const int px = uni ? pm : pn, py = uni ? pn : pm, ss = uni ? 1 : D.n;
    const gcdouble S = as_global(q.ws) + D.offS + (int64_t)(4 * px + 2 * py) * D.nr * D.n + (uni ? (int64_t)a * D.n : a);
    const gcdouble cz = as_global(D.cz) + (int64_t)a * nbp * kzp;
    const int ca = g * 32 + li, cb = ca + 16, la = min(ca, ld - 1) >> 1, lb = min(cb, ld - 1) >> 1;
    const uint32_t os = 8 * ((li & 1) * D.nr * D.n + lk * ss), oa = 8 * (lk * kzp + la), ob = 8 * (lk * kzp + lb);
    f64x4 t0 = F64X4_ZERO, t1 = F64X4_ZERO;
    const Stream x[4] = {{cm, 4, om}, {S, 4 * ss, os}, {cz, 4 * kzp, oa}, {cz, 4 * kzp, ob}};
    staged<4>(x, nb >> 2, [&](int, const double* y) {
        t0 = mfma_f64(y[0], y[2] * y[1], t0);
        t1 = mfma_f64(y[0], y[3] * y[1], t1);
    });
    if (nb & 3) {   // c_m is zero past nb
        const int b0 = nb & ~3, b = min(b0 + lk, nb - 1);
        const double av = load_at(cm + b0, om), h = S[(li & 1) * D.nr * D.n + b * ss];
        t0 = mfma_f64(av, cz[b * kzp + la] * h, t0);
        t1 = mfma_f64(av, cz[b * kzp + lb] * h, t1);
    }
    gdouble out = as_global(q.ws) + D.offG + ((int64_t)(2 * a + pn) * D.km + (pm ? D.kep : 0) + m0) * ld;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = 4 * r + lk;
        if (m0 + m >= kp) continue;
        if (ca < ld) out[m * ld + ca] = t0[r];
        if (cb < ld) out[m * ld + cb] = t1[r];
    }
}

// ---------------------------------------------------------------------------
// Nodes transposed: E = sum_a cos G[a][0], O = sum_a sin G[a][1] at half-axis positions
// (the rows) and 16 columns (m, c); Y[hi] = E + O, Y[lo] = E - O.  A workgroup takes two
// tiles of 16 positions; a wave one of them and half of the nodes.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_nodes_adj_kernel(EwAdj q)
{
    __shared__ double red[2][2][4][64];
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ncols = D.km * D.ld, nap = D.nap, na = D.na, gh = (D.nhNp + 31) >> 5;
    // the groups of positions of one column tile on one XCD, as in the forward
    const int item = blockIdx.x, g = (item >> 3) % gh, cb = ((item >> 3) / gh * 8 + (item & 7)) * 16;
    if (cb >= ncols) return;   // workgroup-uniform
    const int ht = wave & 1, kh = wave >> 1, h0 = min(g * 32 + 16 * ht, D.nhNp - 16), c = cb + li;
    const gcdouble tc = as_global(D.cosN) + (int64_t)h0 * nap, ts = as_global(D.sinN) + (int64_t)h0 * nap;
    const gcdouble G = as_global(q.ws) + D.offG;
    const int full = na >> 2, cc = min(c, ncols - 1);
    const uint32_t ot = 8 * (li * nap + lk), og = 8 * (uint32_t)(2 * lk * ncols + cc);
    f64x4 e = F64X4_ZERO, o = F64X4_ZERO;
    const gcdouble G0 = G + 8 * kh * (int64_t)ncols;   // every other step of four nodes
    const Stream x[4] = {{tc + 4 * kh, 8, ot}, {ts + 4 * kh, 8, ot}, {G0, 16 * (int64_t)ncols, og},
                         {G0 + ncols, 16 * (int64_t)ncols, og}};
    staged<4>(x, (full - kh + 1) >> 1, [&](int, const double* y) {
        e = mfma_f64(y[0], y[2], e);
        o = mfma_f64(y[1], y[3], o);
    });
    if ((na & 3) && kh == (full & 1)) {   // the tables are zero past na
        const int a0 = 4 * full;
        const int64_t a = min(a0 + lk, na - 1);
        e = mfma_f64(load_at(tc + a0, ot), G[2 * a * ncols + cc], e);
        o = mfma_f64(load_at(ts + a0, ot), G[(2 * a + 1) * ncols + cc], o);
    }
    if (kh)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            red[ht][0][r][lane] = e[r];
            red[ht][1][r][lane] = o[r];
        }
    __syncthreads();
    if (kh || c >= ncols || g * 32 + 16 * ht >= D.nhNp) return;
    gdouble out = as_global(q.ws) + D.offY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = h0 + 4 * r + lk, hi = D.nN - 1 - h;
        if (h >= D.nhN) continue;
        const double ev = e[r] + red[ht][0][r][lane], ov = o[r] + red[ht][1][r][lane];
        out[(int64_t)hi * ncols + c] = ev + ov;
        if (hi != h) out[(int64_t)h * ncols + c] = ev - ov;
    }
}

// ---------------------------------------------------------------------------
// Modal transposed: E = sum_{m even} phi_m(h) Y[m], O = the odd modes, at half-axis
// positions (the rows) and 16 columns of one N; Z[hi] = E + O, Z[lo] = E - O.  A
// workgroup takes two tiles of 16 positions; a wave one of them and one parity.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_modal_adj_kernel(EwAdj q)
{
    __shared__ double red[2][4][64];
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, ct = (ld + 15) >> 4, gh = (D.nhMp + 31) >> 5;
    const int item = blockIdx.x, g = (item >> 3) % gh, u = (item >> 3) / gh * 8 + (item & 7);
    const int c = u % ct * 16 + li, N = u / ct;
    if (N >= D.nN) return;   // workgroup-uniform
    const int ht = wave & 1, odd = wave >> 1, h0 = min(g * 32 + 16 * ht, D.nhMp - 16), kt = odd ? D.kot : D.ket;
    const gcdouble y = as_global(q.ws) + D.offY + ((int64_t)N * D.km + (odd ? D.kep : 0)) * ld;
    const gcdouble p = as_global(odd ? D.phio : D.phie) + (int64_t)h0 * kt;
    const uint32_t op = 8 * (li * kt + lk), oy = 8 * (lk * ld + min(c, ld - 1));
    f64x4 t = F64X4_ZERO;
    const Stream x[2] = {{p, 4, op}, {y, 4 * ld, oy}};
    staged<6>(x, (odd ? D.kop : D.kep) >> 2, [&](int, const double* v) { t = mfma_f64(v[0], v[1], t); });
    if (odd)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[ht][r][lane] = t[r];
    __syncthreads();
    if (odd || c >= ld || g * 32 + 16 * ht >= D.nhMp) return;
    const int64_t zs = (int64_t)D.zsM * ld;
    gdouble out = as_global(q.ws) + (int64_t)N * D.zsN * ld + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = h0 + 4 * r + lk, hi = D.nM - 1 - h;
        if (h >= D.nhM) continue;
        const double o = red[ht][r][lane];
        out[hi * zs] = t[r] + o;
        if (hi != h) out[h * zs] = t[r] - o;
    }
}

// ---------------------------------------------------------------------------
// Walk: R = dV exp(-i qc z) sum_l phi_l(z) Z of 16 columns from the matrix instruction
// (rows columns, K the modes, columns the slices) through LDS to the lane that holds the
// slice, then the chain rule along the column.  With P = R T and n = 1 - delta + i beta
// the slice's own terms are -4 P n (real part for delta, imaginary for beta),
// R w = P (n^2 - 1), and sum_{s'>s} R w is the later lanes' plus the lane's own.  T as in
// the scan.
// ---------------------------------------------------------------------------

// The chain rule of a lane's K slices from z on, L lanes to a column; (ur, ui): LDS of
// sum_l phi_l Z, (r0, r1) the rotation at its first slice.  In: carry = sum of R w
// past the round; out: that of the round added.
template <bool MSFT, int K, int L>
__device__ __forceinline__ void ew_chain(const EwDesc& D, const float* d, const float* b, double Sb, double Sd,
                                         double r0, double r1, int z, const double* ur, const double* ui, double* carry,
                                         float* gd, float* gb)
{
    Propagator<MSFT> P;
    P.template start<K>(Sb, Sd, b, d, D.k0dz64, r0, r1, D.step_r, D.step_i);
    const bool density = !MSFT && D.strength == MSFT_STRENGTH_DENSITY;
    const double scale = 2.0 * D.k0dz64;
    double vd[K], vb[K], wr = 0.0, wi = 0.0;   // the slices' own terms; sum of R w so far
    auto slices = [&](auto small) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double xr = ur[slice_row(z + k)], xi = ui[slice_row(z + k)], dk = d[k], bk = b[k], nr = 1.0 - dk;
            const double pr = xr * P.tr - xi * P.ti, pi = xr * P.ti + xi * P.tr;
            vd[k] = -4.0 * (pr * nr - pi * bk);
            vb[k] = -4.0 * (pr * bk + pi * nr);
            if (density) {
                vd[k] = 2.0 * pr;
                vb[k] = -2.0 * pi;
            }
            if (MSFT) {
                const double chr = dk * (dk - 2.0) - bk * bk, chi = 2.0 * bk * nr;
                wr += pr * chr - pi * chi;
                wi += pr * chi + pi * chr;
                // what follows the slice is the sum past the lane's last, less what the lane had here
                vd[k] -= scale * wi;
                vb[k] += scale * wr;
            }
            if (k + 1 < K) P.template next<decltype(small)::value>(bk, dk);
        }
    };
    if (!MSFT || P.small) slices(std::true_type{});
    else slices(std::false_type{});
    double er = 0.0, ei = 0.0;
    if (MSFT) {
        const double qr = group_prefix_f64<L>(wr), qi = group_prefix_f64<L>(wi);
        const double sr = group_last_f64<L>(qr), si = group_last_f64<L>(qi);
        er = scale * ((carry[0] + (sr - qr)) + wr);
        ei = scale * ((carry[1] + (si - qi)) + wi);
        carry[0] += sr;
        carry[1] += si;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        gd[k] = (float)(vd[k] + ei);
        gb[k] = (float)(vb[k] - er);
    }
}

template <int K>
__device__ __forceinline__ void store_slices(float* od, float* ob, int z, int nz, const float* gd, const float* gb)
{
    if (K % 4 == 0 && (nz & 3) == 0) {
#pragma unroll
        for (int k = 0; k + 3 < K; k += 4)
            if (z + k < nz) {
                *(float4*)(od + z + k) = make_float4(gd[k], gd[k + 1], gd[k + 2], gd[k + 3]);
                *(float4*)(ob + z + k) = make_float4(gb[k], gb[k + 1], gb[k + 2], gb[k + 3]);
            }
        return;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (z + k < nz) {
            od[z + k] = gd[k];
            ob[z + k] = gb[k];
        }
}

// Whole columns: even and odd modes on the half axis, E + O and E - O the mirror slices.  The
// products' rows are 16 columns, Re and Im apart, or 8 columns' (Re, Im).  A wave takes every
// fourth (Re or Im and every other) tile of 16 half-axis slices, at most two, both against one
// operand; 16 modes of each parity at a time, all their loads ahead of the products.
template <bool MSFT, int COLS, int K>
__global__ __launch_bounds__(EA_THREADS, K == 8 ? 3 : 4) void ew_walk_kernel(EwAdj q)
{
    constexpr int L = EA_THREADS / COLS, NZ = L * K;
    __shared__ double sm[COLS == 16 ? 2 * slice_row(16 * K) : slice_row(32 * K)];   // Re and Im of 16 lanes' slices, or 32 lanes'
    const EwDesc& D = *q.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int cl = tid / L, z0 = tid % L * K, nz = D.nz;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)blockIdx.x * COLS;
    const bool in = c0 + cl < ncol;
    const int64_t off = (in ? c0 + cl : ncol - 1) * nz;
    float d[K], b[K];
    load_slices<K>(q.delta + off, q.beta + off, z0, nz, in, d, b);
    const gcdouble rot = as_global(D.rot) + 2 * min(z0, (nz + EW_ZC - 1) / EW_ZC * EW_ZC - 1);
    const double r0 = rot[0], r1 = rot[1];
    // slices past the column's end
    for (int k = slice_row(nz) + tid; k < slice_row(NZ); k += EA_THREADS) {
        sm[k] = 0.0;
        if (COLS == 16) sm[slice_row(NZ) + k] = 0.0;
    }
    {
        const int set = COLS == 16 ? wave & 1 : 0, nh = (nz + 1) >> 1, kze = D.kze, kzo = D.kz - kze, last = D.kzp - 1;
        const int col = COLS == 16 ? li : li >> 1, ri = COLS == 16 ? set : li & 1;
        const int h0 = COLS == 16 ? 16 * (wave >> 1) : 16 * wave, h1 = h0 + (COLS == 16 ? 32 : 64);
        const uint32_t oz = 8 * (uint32_t)((min(c0 + col, ncol - 1) - c0) * D.ld);
        const double sign = ri ? -1.0 : 1.0;   // -i of the odd modes: (im, -re)
        const gcdouble z = as_global(q.ws) + c0 * D.ld;
        const int a0 = h0 < nh ? h0 : 0, a1 = h1 < nh ? h1 : a0;   // a tile past the middle is not stored
        const gcdouble e0 = as_global(D.phize) + (int64_t)a0 * D.kzet, e1 = as_global(D.phize) + (int64_t)a1 * D.kzet;
        const gcdouble o0 = as_global(D.phizo) + (int64_t)a0 * D.kzot, o1 = as_global(D.phizo) + (int64_t)a1 * D.kzot;
        const uint32_t oe = 8 * (li * D.kzet + lk), oo = 8 * (li * D.kzot + lk);
        f64x4 te[2] = {F64X4_ZERO, F64X4_ZERO}, to[2] = {F64X4_ZERO, F64X4_ZERO};
        for (int l0 = 0; l0 < max(kze, kzo); l0 += 16) {
            // the half-axis modes are zero past their last; what they meet there is finite
            double x[4][6];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int le = l0 < D.kzet ? l0 + 4 * u : 0, lo = l0 < D.kzot ? l0 + 4 * u : 0;
                x[u][0] = load_at(z, oz + 8 * (2 * min(le + lk, last) + ri));
                x[u][1] = load_at(z, oz + 8 * (2 * min(kze + lo + lk, last) + 1 - ri));
                x[u][2] = load_at(e0 + le, oe);
                x[u][3] = load_at(e1 + le, oe);
                x[u][4] = load_at(o0 + lo, oo);
                x[u][5] = load_at(o1 + lo, oo);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (l0 + 4 * u < kze) {
                    te[0] = mfma_f64(x[u][0], x[u][2], te[0]);
                    te[1] = mfma_f64(x[u][0], x[u][3], te[1]);
                }
                if (l0 + 4 * u < kzo) {
                    const double v = sign * x[u][1];
                    to[0] = mfma_f64(v, x[u][4], to[0]);
                    to[1] = mfma_f64(v, x[u][5], to[1]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int h = (k ? h1 : h0) + li;
            if (h < nh) {
                double* hi = sm + set * slice_row(NZ) + slice_row(nz - 1 - h) + lk;
                double* lo = sm + set * slice_row(NZ) + slice_row(h) + lk;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    lo[4 * r] = te[k][r] - to[k][r];
                    hi[4 * r] = te[k][r] + to[k][r];   // an odd column's middle: the odd part is zero
                }
            }
        }
    }
    double Sb = 0.0, Sd = 0.0;
    if (MSFT) {
        double sb = 0.0, sd = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sb += (double)b[k];
            sd += (double)d[k];
        }
        Sb = group_prefix_f64<L>(sb) - sb;
        Sd = group_prefix_f64<L>(sd) - sd;
    }
    __syncthreads();
    double carry[2] = {0.0, 0.0};
    float gd[K], gb[K];
    const double* u = sm + (COLS == 16 ? cl : 2 * cl);
    ew_chain<MSFT, K, L>(D, d, b, Sb, Sd, r0, r1, z0, u, u + (COLS == 16 ? slice_row(NZ) : 1), carry, gd, gb);
    if (in) store_slices<K>(q.grad_delta + off, q.grad_beta + off, z0, nz, gd, gb);
}

// Longer columns, in rounds of 64 slices from the exit face back, after a pass that sums
// beta + i delta of each round.
constexpr int EA_ROUNDS = 4096 / EW_ZC;

template <bool MSFT>
__global__ __launch_bounds__(EA_THREADS) void ew_walk_rounds_kernel(EwAdj q)
{
    __shared__ double sm[2 * slice_row(EW_ZC)];
    __shared__ double pre[2 * EA_ROUNDS * EW_COLS];   // beta, delta before each round
    const EwDesc& D = *q.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int cl = tid >> 4, zl = (tid & 15) * 4, nz = D.nz, kzt = D.kzt, kze = D.kze;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)blockIdx.x * EW_COLS;
    const bool in = c0 + cl < ncol;
    const int64_t off = (in ? c0 + cl : ncol - 1) * nz;
    const int rounds = (nz + EW_ZC - 1) / EW_ZC;
    float d[4], b[4];
    if (MSFT) {
        double tb = 0.0, td = 0.0;
        for (int r = 0; r < rounds; ++r) {
            if ((tid & 15) == 0) {
                pre[(2 * r) * EW_COLS + cl] = tb;
                pre[(2 * r + 1) * EW_COLS + cl] = td;
            }
            if (r + 1 == rounds) break;
            load_slices<4>(q.delta + off, q.beta + off, r * EW_ZC + zl, nz, in, d, b);
            tb += row_last_f64(row_prefix_f64(((double)b[0] + b[1]) + ((double)b[2] + b[3])));
            td += row_last_f64(row_prefix_f64(((double)d[0] + d[1]) + ((double)d[2] + d[3])));
        }
    }
    const int ri = wave & 1, zt = (wave >> 1) * 32;
    const double* zh = q.ws + min(c0 + li, ncol - 1) * D.ld;
    const gcdouble rot = as_global(D.rot) + 2 * zl;
    double carry[2] = {0.0, 0.0};
    for (int rd = rounds - 1; rd >= 0; --rd) {
        const int z0 = rd * EW_ZC;
        load_slices<4>(q.delta + off, q.beta + off, z0 + zl, nz, in, d, b);
        {
            f64x4 t0 = F64X4_ZERO, t1 = F64X4_ZERO;
            const gcdouble p = as_global(D.phiz) + (int64_t)(z0 + zt + li) * kzt;
            for_steps<4>(D.kzp / 4, [&](int ks) {
                const int l = 4 * ks + lk;
                const bool odd = l >= kze;   // -i of the odd modes: (im, -re)
                double v = zh[2 * l + (odd ? 1 - ri : ri)];
                if (odd && ri) v = -v;
                t0 = mfma_f64(v, p[l], t0);
                t1 = mfma_f64(v, p[16 * kzt + l], t1);
            });
            double* o = sm + ri * slice_row(EW_ZC) + slice_row(zt + li) + lk;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[4 * r] = t0[r];
                o[slice_row(16) + 4 * r] = t1[r];
            }
        }
        __syncthreads();
        double Sb = 0.0, Sd = 0.0;
        if (MSFT) {
            const double sb = ((double)b[0] + b[1]) + ((double)b[2] + b[3]);
            const double sd = ((double)d[0] + d[1]) + ((double)d[2] + d[3]);
            Sb = pre[2 * rd * EW_COLS + cl] + (row_prefix_f64(sb) - sb);
            Sd = pre[(2 * rd + 1) * EW_COLS + cl] + (row_prefix_f64(sd) - sd);
        }
        float gd[4], gb[4];
        ew_chain<MSFT, 4, 16>(D, d, b, Sb, Sd, rot[2 * z0], rot[2 * z0 + 1], zl, sm + cl, sm + slice_row(EW_ZC) + cl,
                              carry, gd, gb);
        if (in) store_slices<4>(q.grad_delta + off, q.grad_beta + off, z0 + zl, nz, gd, gb);
        __syncthreads();   // the next round rewrites sm
    }
}

template <bool MSFT>
void launch_walk(const EwAdj& a, const EwDesc& d, hipStream_t s)
{
    const dim3 grid((unsigned)ceil_div((int64_t)d.nx * d.ny, ew_columns(d.nz))), th(EA_THREADS);
    switch (ew_rounds(d.nz)) {
    case 1: hipLaunchKernelGGL((ew_walk_kernel<MSFT, 16, 4>), grid, th, 0, s, a); break;
    case 2: hipLaunchKernelGGL((ew_walk_kernel<MSFT, 16, 8>), grid, th, 0, s, a); break;
    case 3: hipLaunchKernelGGL((ew_walk_kernel<MSFT, 8, 6>), grid, th, 0, s, a); break;
    case 4: hipLaunchKernelGGL((ew_walk_kernel<MSFT, 8, 8>), grid, th, 0, s, a); break;
    default: hipLaunchKernelGGL(ew_walk_rounds_kernel<MSFT>, grid, th, 0, s, a);
    }
}

}  // namespace

int launch_ew_adjoint(const EwAdj& a, const EwDesc& d, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    auto launch = [&](auto kernel, int64_t blocks, int threads, size_t lds) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(threads), lds, s, a);
    };
    // `inner` workgroups of each of `outer` units on one XCD
    auto on_xcd = [](int64_t outer, int64_t inner) { return ceil_div(outer, 8) * 8 * inner; };
    launch(ew_rows_kernel, d.rows, EA_THREADS, 0);
    launch(ew_coef_adj_kernel, d.nrp / 16 * 8, CA_THREADS, d.n * 17 * sizeof(double));
    launch(ew_yz_adj_kernel, on_xcd(d.na, 2 * ceil_div(d.kep > d.kop ? d.kep : d.kop, 32) * ceil_div(d.ld, 32)),
           EA_THREADS, 0);
    launch(ew_nodes_adj_kernel, on_xcd(ceil_div((int64_t)d.km * d.ld, 16), ceil_div(d.nhNp, 32)), EA_THREADS, 0);
    launch(ew_modal_adj_kernel, on_xcd(ceil_div(d.ld, 16) * d.nN, ceil_div(d.nhMp, 32)), EA_THREADS, 0);
    if (d.strength == MSFT_STRENGTH_MSFT) launch_walk<true>(a, d, s);
    else launch_walk<false>(a, d, s);
    return (int)hipGetLastError();
}

}  // namespace msft
