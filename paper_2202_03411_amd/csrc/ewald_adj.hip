// Adjoint of the spherical-coordinate forward model (see ewald.h): the five stages of
// the forward transposed, in FP64, and the column walk of the chain rule.
//
//   rows   H(row, k)  = sum over the row's pixels of T_k(t) h     (h = g conj(A), folded
//          over the four mirror pixels), then node values' gradients
//   yz     Gh[a]      = sum_b c_m(a, b) c_l(a, b) H(a, b)
//   nodes  Yh[N]      = sum_a {cos, sin}(q_N(a) N) Gh[a]
//   modal  Zh[N][M]   = sum_m phi_m(M) Yh[N]
//   walk   R(z)       = exp(-i qc z) sum_l phi_l(z) Zh, then along each column
//          dL/d delta, dL/d beta from R (Eqs. (7)-(9))
#include <hip/hip_runtime.h>

#include "ewald.h"
#include "msft_internal.h"
#include "wave_f64.h"

namespace msft {

namespace {

constexpr int EA_THREADS = 256;   // of a workgroup, but for the rows of more than 256 nodes: 128
constexpr int EA_WAVES = EA_THREADS / 64;

// Sums of eight values over a wave: two exchange steps leave a lane two of the eight
// (indices 4 bit0(lane) + 2 bit1(lane) + {0, 1}), which are then summed over the lanes
// of the same two bits.
__device__ __forceinline__ void wave_sum8(const double* v, int lane, double* out)
{
    const bool b0 = lane & 1, b1 = lane & 2;
    double w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double keep = b0 ? v[4 + k] : v[k], send = b0 ? v[k] : v[4 + k];
        w[k] = keep + dpp_f64<0xB1, 0xF>(send);   // quad_perm 1,0,3,2
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double keep = b1 ? w[2 + k] : w[k], send = b1 ? w[k] : w[2 + k];
        double s = keep + dpp_f64<0x4E, 0xF>(send);   // quad_perm 2,3,0,1
        s += dpp_f64<0x124, 0xF>(s);                  // row_ror 4
        s += dpp_f64<0x128, 0xF>(s);                  // row_ror 8
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        out[k] = s;
    }
}

// ---------------------------------------------------------------------------
// Rows: one workgroup per pixel row.  A thread folds h of its columns' mirror pixels
// into the eight parts, runs the Chebyshev recurrences and, for every k, the workgroup
// sums T_k times the parts over the row; the sums go through LDS to the transposed
// node transform.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_rows_kernel(EwAdj q)
{
    extern __shared__ double lds[];   // [waves][n][8]
    const EwDesc& D = *q.d;
    const int n = D.n, N = D.det_n, half = D.rows, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = blockIdx.x, jh = N - 1 - j, threads = blockDim.x;
    double* part = lds + (size_t)wave * n * 8;
    for (int k = lane; k < n * 8; k += 64) part[k] = 0.0;
    __syncthreads();
    const float2* A = (const float2*)q.amplitude;
    for (int i0 = 0; i0 < half; i0 += threads) {
        const int i = i0 + tid;
        double H[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) H[c] = 0.0;
        double t = 0.0;
        if (i < half) {
            t = D.tq[(int64_t)j * half + i];
            const bool rim = !(t == t);
            if (rim) t = 0.0;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const bool px = !(m & 1), py = !(m & 2);
                const int ii = px ? N - 1 - i : i, jj = py ? jh : j;
                if (rim || (!px && ii == N - 1 - i) || (!py && jj == jh)) continue;
                const double sx = px ? 1.0 : -1.0, sy = py ? 1.0 : -1.0;
                const int64_t p = (int64_t)jj * N + ii;
                const double g = (double)q.grad_intensity[p];
                const float2 a = A[p];
                const double hr = g * (double)a.x, hi = -g * (double)a.y;
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
        }
        const double x2 = 2.0 * (2.0 * t * t - 1.0);
        double e0 = 1.0, e1 = 0.5 * x2, o0 = t, o1 = (x2 - 1.0) * t;
        for (int k = 0; k < n; ++k) {
            double v[8], s[2];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                v[c] = e0 * H[c];
                v[4 + c] = o0 * H[4 + c];
            }
            wave_sum8(v, lane, s);
            if (lane < 4) {
                double* out = part + k * 8 + 4 * (lane & 1) + (lane & 2);
                out[0] += s[0];
                out[1] += s[1];
            }
            const double e2 = x2 * e1 - e0, o2 = x2 * o1 - o0;
            e0 = e1;
            e1 = e2;
            o0 = o1;
            o1 = o2;
        }
    }
    __syncthreads();
    for (int k = tid; k < n * 8; k += threads) {
        double s = lds[k];
        for (int w = 1; w < threads >> 6; ++w) s += lds[(size_t)w * n * 8 + k];
        lds[k] = s;
    }
    __syncthreads();
    double* out = q.ws + D.offA + (int64_t)j * n * 8;
    for (int o = tid; o < n * 8; o += threads) {
        const int comp = o & 7, a = o >> 3;
        const double* m = (comp & 4 ? D.dcto : D.dcte) + (size_t)a * n;
        double s = 0.0;
#pragma unroll 4
        for (int k = 0; k < n; ++k) s += m[k] * lds[k * 8 + comp];
        out[o] = s;
    }
}

// ---------------------------------------------------------------------------
// yz transposed: Gh[a][pN][m][(l, ri)] = sum_b c_m(a, b) c_l(a, b) H(a, b)[pN][pM(m)][ri].
// A wave takes one a, one pN, 16 modes m of a parity (the rows) and up to four tiles of
// 16 columns (l, ri); K runs over b, the second operand formed from c_l and H.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_yz_adj_kernel(EwAdj q)
{
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int te = (D.kep + 15) >> 4, to = (D.kop + 15) >> 4, cg = (D.ld + 63) >> 6;
    int64_t u = (int64_t)blockIdx.x * EA_WAVES + (threadIdx.x >> 6);
    const int g = (int)(u % cg);
    u /= cg;
    const int mt = (int)(u % (te + to));
    u /= te + to;
    const int pn = (int)(u & 1), a = (int)(u >> 1);
    if (a >= D.na) return;
    const int pm = mt >= te, m0 = (pm ? mt - te : mt) * 16, kp = pm ? D.kop : D.kep;
    const int nbp = D.nbp, kzp = D.kzp, nb = D.nb, ld = D.ld;
    // rows beyond the parity's modes read its last row and are not stored
    const double* cm = D.cm + ((size_t)a * D.km + (pm ? D.kep : 0) + min(m0 + li, kp - 1)) * nbp + lk;
    const int px = D.uniform ? pm : pn, py = D.uniform ? pn : pm;
    const double* H = q.ws + D.offA + 4 * px + 2 * py + (li & 1);
    const int64_t hs = D.uniform ? 8 : (int64_t)D.n * 8, ha = D.uniform ? (int64_t)D.n * 8 : 8;
    H += a * ha;
    f64x4 acc[4];
    int lz[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        lz[t] = min(g * 64 + t * 16 + li, ld - 1) >> 1;
    }
    const int nt = min(4, (ld - g * 64 + 15) >> 4);
    for_steps<2>(nbp / 4, [&](int ks) {
        const int b = 4 * ks + lk, bc = min(b, nb - 1);
        const double av = cm[4 * ks], h = H[bc * hs];   // cm is zero for b >= nb
        const double* cz = D.cz + ((size_t)a * nbp + bc) * kzp;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (t < nt) acc[t] = mfma_f64(av, cz[lz[t]] * h, acc[t]);
    });
    double* out = q.ws + D.offG + ((int64_t)(2 * a + pn) * D.km + (pm ? D.kep : 0)) * ld;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int c = g * 64 + t * 16 + li;
        if (t >= nt || c >= ld) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 4 * r + lk;
            if (m < kp) out[(int64_t)m * ld + c] = acc[t][r];
        }
    }
}

// ---------------------------------------------------------------------------
// Nodes transposed: E = sum_a cos Gh[a][0], O = sum_a sin Gh[a][1] at 16 half-axis
// positions (the rows) and 16 columns (m, c); Yh[hi] = E + O, Yh[lo] = E - O.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_nodes_adj_kernel(EwAdj q)
{
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int ncols = D.km * D.ld, ct = (ncols + 15) >> 4, nap = D.nap, gh = (D.nhNp + 31) >> 5;
    const int64_t u = (int64_t)blockIdx.x * EA_WAVES + (threadIdx.x >> 6);
    const int c = (int)(u % ct) * 16 + li, g = (int)(u / ct);
    if (g >= gh) return;
    const bool two = g * 32 + 16 < D.nhNp;
    const size_t at = (size_t)(g * 32 + li) * nap + lk;
    const double* tc = D.cosN + at;
    const double* ts = D.sinN + at;
    const int64_t step16 = two ? (int64_t)16 * nap : 0;
    const double* G = q.ws + D.offG + min(c, ncols - 1);
    f64x4 e0 = {0.0, 0.0, 0.0, 0.0}, e1 = e0, o0 = e0, o1 = e0;
    for_steps<4>(nap / 4, [&](int ks) {
        const int a = min(4 * ks + lk, D.na - 1);   // the tables are zero beyond na
        const double ge = G[(int64_t)(2 * a) * ncols], go = G[(int64_t)(2 * a + 1) * ncols];
        e0 = mfma_f64(tc[4 * ks], ge, e0);
        o0 = mfma_f64(ts[4 * ks], go, o0);
        if (two) {
            e1 = mfma_f64(tc[step16 + 4 * ks], ge, e1);
            o1 = mfma_f64(ts[step16 + 4 * ks], go, o1);
        }
    });
    if (c >= ncols) return;
    double* out = q.ws + D.offY + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = g * 32 + 4 * r + lk;
        if (h < D.nhN) {
            out[(int64_t)(D.nN - 1 - h) * ncols] = e0[r] + o0[r];
            if (D.nN - 1 - h != h) out[(int64_t)h * ncols] = e0[r] - o0[r];
        }
        if (two && h + 16 < D.nhN) {
            const int k = h + 16;
            out[(int64_t)(D.nN - 1 - k) * ncols] = e1[r] + o1[r];
            if (D.nN - 1 - k != k) out[(int64_t)k * ncols] = e1[r] - o1[r];
        }
    }
}

// ---------------------------------------------------------------------------
// Modal transposed: E = sum_{m even} phi_m(h) Yh[m], O = the odd modes, at 16 half-axis
// positions and 16 columns of one N; Zh[hi] = E + O, Zh[lo] = E - O.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(EA_THREADS) void ew_modal_adj_kernel(EwAdj q)
{
    const EwDesc& D = *q.d;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, ct = (ld + 15) >> 4, gh = (D.nhMp + 31) >> 5;
    int64_t u = (int64_t)blockIdx.x * EA_WAVES + (threadIdx.x >> 6);
    const int g = (int)(u % gh);
    u /= gh;
    const int c = (int)(u % ct) * 16 + li, N = (int)(u / ct);
    if (N >= D.nN) return;
    const bool two = g * 32 + 16 < D.nhMp;
    const double* y = q.ws + D.offY + ((int64_t)N * D.km + lk) * ld + min(c, ld - 1);
    const double* pe = D.phie + (size_t)(g * 32 + li) * D.ket + lk;
    const double* po = D.phio + (size_t)(g * 32 + li) * D.kot + lk;
    const int64_t se = two ? (int64_t)16 * D.ket : 0, so = two ? (int64_t)16 * D.kot : 0;
    f64x4 e0 = {0.0, 0.0, 0.0, 0.0}, e1 = e0, o0 = e0, o1 = e0;
    for_steps<3>(D.kep / 4, [&](int ks) {
        const double v = y[(int64_t)4 * ks * ld];
        e0 = mfma_f64(pe[4 * ks], v, e0);
        if (two) e1 = mfma_f64(pe[se + 4 * ks], v, e1);
    });
    y += (int64_t)D.kep * ld;
    for_steps<3>(D.kop / 4, [&](int ks) {
        const double v = y[(int64_t)4 * ks * ld];
        o0 = mfma_f64(po[4 * ks], v, o0);
        if (two) o1 = mfma_f64(po[so + 4 * ks], v, o1);
    });
    if (c >= ld) return;
    const int64_t zs = (int64_t)D.zsM * ld;
    double* out = q.ws + (int64_t)N * D.zsN * ld + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int h = g * 32 + 4 * r + lk;
        if (h < D.nhM) {
            out[(D.nM - 1 - h) * zs] = e0[r] + o0[r];
            if (D.nM - 1 - h != h) out[h * zs] = e0[r] - o0[r];
        }
        if (two && h + 16 < D.nhM) {
            const int k = h + 16;
            out[(D.nM - 1 - k) * zs] = e1[r] + o1[r];
            if (D.nM - 1 - k != k) out[k * zs] = e1[r] - o1[r];
        }
    }
}

// ---------------------------------------------------------------------------
// Walk: 16 columns, rounds of EW_ZC slices from the exit face back.  A first pass sums
// beta + i delta of each round (the exclusive prefix S of a round's first slice); then,
// round by round, R = exp(-i qc z) sum_l phi_l(z) Zh comes from the matrix instruction
// (rows columns, K the modes, columns the slices) through LDS to the thread that holds
// the slice, and sum_{s'>s} R w accumulates on the way.  FP64, T in FP32 as the scan
// forms it.
// ---------------------------------------------------------------------------
constexpr int EA_LD = EW_COLS + 1;
constexpr int EA_ROUNDS = 4096 / EW_ZC;

__global__ __launch_bounds__(EA_THREADS) void ew_walk_kernel(EwAdj q)
{
    __shared__ double sm[2][EW_ZC * EA_LD];
    __shared__ double pre[2][EA_ROUNDS][EW_COLS];   // beta, delta before each round
    const EwDesc& D = *q.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cl = tid >> 4, zl = (tid & 15) * 4, nz = D.nz, strength = D.strength;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)blockIdx.x * EW_COLS;
    const bool in = c0 + cl < ncol;
    const int64_t col = in ? c0 + cl : ncol - 1;
    const float* dc = q.delta + col * nz;
    const float* bc = q.beta + col * nz;
    const bool vec = (nz & 3) == 0;
    const int rounds = (nz + EW_ZC - 1) / EW_ZC;
    float d[4], b[4];
    auto load = [&](int z) {
        if (in && vec && z < nz) {
            const float4 dv = *(const float4*)(dc + z), bv = *(const float4*)(bc + z);
            d[0] = dv.x; d[1] = dv.y; d[2] = dv.z; d[3] = dv.w;
            b[0] = bv.x; b[1] = bv.y; b[2] = bv.z; b[3] = bv.w;
            return;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool ok = in && z + k < nz;
            d[k] = ok ? dc[z + k] : 0.0f;
            b[k] = ok ? bc[z + k] : 0.0f;
        }
    };
    if (strength == MSFT_STRENGTH_MSFT) {
        double tb = 0.0, td = 0.0;
        for (int r = 0; r + 1 < rounds; ++r) {
            load(r * EW_ZC + zl);
            if ((tid & 15) == 0) {
                pre[0][r][cl] = tb;
                pre[1][r][cl] = td;
            }
            tb += row_last_f64(row_prefix_f64(((double)b[0] + b[1]) + ((double)b[2] + b[3])));
            td += row_last_f64(row_prefix_f64(((double)d[0] + d[1]) + ((double)d[2] + d[3])));
        }
        if ((tid & 15) == 0) {
            pre[0][rounds - 1][cl] = tb;
            pre[1][rounds - 1][cl] = td;
        }
    }
    const double dV = D.dV64, k0dz = D.k0dz64;
    const int ri = wave & 1, zt = (wave >> 1) * 32;
    const double* zh = q.ws + min(c0 + (lane & 15), ncol - 1) * D.ld;
    double carry_r = 0.0, carry_i = 0.0;
    for (int rd = rounds - 1; rd >= 0; --rd) {
        const int z0 = rd * EW_ZC;
        load(z0 + zl);
        {
            f64x4 r0 = {0.0, 0.0, 0.0, 0.0}, r1 = r0;
            const double* p = D.phiz + (size_t)(z0 + zt + (lane & 15)) * D.kzt;
            for_steps<2>(D.kzp / 4, [&](int ks) {
                const int l = 4 * ks + (lane >> 4);
                const bool odd = l >= D.kze;   // -i of the odd modes: (im, -re)
                double v = zh[2 * l + (odd ? 1 - ri : ri)];
                if (odd && ri) v = -v;
                r0 = mfma_f64(v, p[l], r0);
                r1 = mfma_f64(v, p[(size_t)16 * D.kzt + l], r1);
            });
            double* o = sm[ri] + (zt + (lane & 15)) * EA_LD + (lane >> 4);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[4 * r] = r0[r];
                o[16 * EA_LD + 4 * r] = r1[r];
            }
        }
        __syncthreads();
        double gd[4], gb[4], rwr[4], rwi[4];
        double Sb = 0.0, Sd = 0.0;
        if (strength == MSFT_STRENGTH_MSFT) {
            const double sb = ((double)b[0] + b[1]) + ((double)b[2] + b[3]);
            const double sd = ((double)d[0] + d[1]) + ((double)d[2] + d[3]);
            Sb = pre[0][rd][cl] + (row_prefix_f64(sb) - sb);
            Sd = pre[1][rd][cl] + (row_prefix_f64(sd) - sd);
        }
        const double2* rot = (const double2*)D.rot + z0 + zl;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double ur = sm[0][(zl + k) * EA_LD + cl], ui = sm[1][(zl + k) * EA_LD + cl];
            const double2 e = rot[k];
            const double rr = ur * e.x - ui * e.y, rim = ur * e.y + ui * e.x;
            rwr[k] = rwi[k] = 0.0;
            if (strength == MSFT_STRENGTH_DENSITY) {
                gd[k] = 2.0 * dV * rr;
                gb[k] = -2.0 * dV * rim;
                continue;
            }
            const double dd = d[k], bb = b[k];
            double tr = 1.0, ti = 0.0;
            if (strength == MSFT_STRENGTH_MSFT) {
                constexpr double kTwoPi = 6.283185307179586476925286766559;
                const double ph = -k0dz * Sd;
                const float mag = expf((float)(-k0dz * Sb));
                float sn, cs;
                sincosf((float)(ph - kTwoPi * rint(ph * (1.0 / kTwoPi))), &sn, &cs);
                tr = (double)mag * (double)cs;
                ti = (double)mag * (double)sn;
            }
            // dw/d delta = dV T (-2 n), dw/d beta = dV T (2 i n), n = 1 - delta + i beta
            const double nr = 1.0 - dd;
            const double xr = 2.0 * dV * (tr * nr - ti * bb), xi = 2.0 * dV * (tr * bb + ti * nr);
            gd[k] = -2.0 * (rr * xr - rim * xi);
            gb[k] = -2.0 * (rr * xi + rim * xr);
            if (strength == MSFT_STRENGTH_MSFT) {
                const double chr = dd * (dd - 2.0) - bb * bb, chi = 2.0 * bb * (1.0 - dd);
                const double wr = dV * (chr * tr - chi * ti), wi = dV * (chr * ti + chi * tr);
                rwr[k] = rr * wr - rim * wi;
                rwi[k] = rr * wi + rim * wr;
                Sb += bb;
                Sd += dd;
            }
        }
        if (strength == MSFT_STRENGTH_MSFT) {
            const double lr = (rwr[0] + rwr[1]) + (rwr[2] + rwr[3]), im = (rwi[0] + rwi[1]) + (rwi[2] + rwi[3]);
            const double pr = row_prefix_f64(lr), pi = row_prefix_f64(im);
            const double tr = row_last_f64(pr), ti = row_last_f64(pi);
            double er = carry_r + (tr - pr), ei = carry_i + (ti - pi);   // later lanes and rounds
#pragma unroll
            for (int k = 3; k >= 0; --k) {
                gd[k] += 2.0 * k0dz * ei;
                gb[k] -= 2.0 * k0dz * er;
                er += rwr[k];
                ei += rwi[k];
            }
            carry_r += tr;
            carry_i += ti;
        }
        float* od = q.grad_delta + col * nz + z0 + zl;
        float* ob = q.grad_beta + col * nz + z0 + zl;
        if (in && vec && z0 + zl < nz) {
            *(float4*)od = make_float4((float)gd[0], (float)gd[1], (float)gd[2], (float)gd[3]);
            *(float4*)ob = make_float4((float)gb[0], (float)gb[1], (float)gb[2], (float)gb[3]);
        } else if (in) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (z0 + zl + k < nz) {
                    od[k] = (float)gd[k];
                    ob[k] = (float)gb[k];
                }
        }
        __syncthreads();   // the next round rewrites sm
    }
}

}  // namespace

int launch_ew_adjoint(const EwAdj& a, const EwDesc& d, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    auto blocks = [](int64_t waves) { return dim3((unsigned)ceil_div(waves, EA_WAVES)); };
    const dim3 th(EA_THREADS);
    // a wave's sums are 64 n bytes of LDS: four waves up to 256 nodes, two up to the limit of 512
    const int rw = d.n <= 256 ? EA_WAVES : 2;
    hipLaunchKernelGGL(ew_rows_kernel, dim3(d.rows), dim3(64 * rw), d.n * 8 * rw * sizeof(double), s, a);
    const int64_t mt = ceil_div(d.kep, 16) + ceil_div(d.kop, 16);
    hipLaunchKernelGGL(ew_yz_adj_kernel, blocks(2 * d.na * mt * ceil_div(d.ld, 64)), th, 0, s, a);
    hipLaunchKernelGGL(ew_nodes_adj_kernel,
                       blocks(ceil_div((int64_t)d.km * d.ld, 16) * ceil_div(d.nhNp, 32)), th, 0, s, a);
    hipLaunchKernelGGL(ew_modal_adj_kernel, blocks(ceil_div(d.ld, 16) * ceil_div(d.nhMp, 32) * d.nN), th, 0, s, a);
    hipLaunchKernelGGL(ew_walk_kernel, dim3((unsigned)ceil_div((int64_t)d.nx * d.ny, EW_COLS)), th, 0, s, a);
    return (int)hipGetLastError();
}

}  // namespace msft
