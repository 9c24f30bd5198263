// Forward model in spherical coordinates about a detector axis (see ewald.h): the
// column scan with its projection on the z modes, three contractions on the FP64 matrix
// instruction, and the evaluation of each pixel row's Chebyshev series.
//
// The FP64 matrix instruction runs at the FP64 vector rate (78.6 TFLOP/s), one
// 16 x 16 x 4 product in 64 cycles of a SIMD, so its operands can come from the L1 cache
// without staging: one operand of 512 bytes a product.  At the sizes of a pattern
// (128^3 voxels, 512^2 pixels) a whole call is some 0.3 G multiply-adds, and the six
// launches are bound by their own latency and by reading delta and beta once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ewald.h"
#include "msft_internal.h"
#include "wave_f64.h"

namespace msft {

namespace {

constexpr int EW_THREADS = 256;

// The request a workgroup belongs to and its index within it.  The kernels take one request
// (72 bytes of arguments: 2.7 us a launch on the host) or a batch (1.5 KB: 4.0 us); the scan,
// whose many workgroups would each wait for the sizes and table pointers first, has them
// among the arguments (192^3: 39.3 -> 36.7 us; the other kernels gain nothing by it).
__device__ __forceinline__ const EwReq& ew_request(const EwBatch& b, int& item)
{
    int r = 0;
    while (r + 1 < b.n && (int)blockIdx.x >= b.begin[r + 1]) ++r;
    item = (int)blockIdx.x - b.begin[r];
    return b.req[r];
}
__device__ __forceinline__ const EwReq& ew_request(const EwReq& r, int& item)
{
    item = (int)blockIdx.x;
    return r;
}
__device__ __forceinline__ const EwReq& ew_request(const EwOne& r, int& item)
{
    item = (int)blockIdx.x;
    return r.req;
}
template <typename A>
__device__ __forceinline__ const EwDesc& ew_desc(const A&, const EwReq& q) { return *q.d; }
__device__ __forceinline__ const EwDesc& ew_desc(const EwOne& r, const EwReq&) { return r.d; }

// ---------------------------------------------------------------------------
// Scan: w of 16 columns and Z_l = sum_z phi_l(z) exp(-i qc z) w.
//
// The 16 lanes of a column hold K consecutive slices each.  The exclusive prefix
// S = sum_{s'<s} (beta + i delta) is the carry of earlier rounds plus a DPP prefix over
// the column's lanes; T = exp(-k0 dz S) is evaluated in full at a lane's first slice and
// by the slices' own factors after it.  dV times the rotated w goes to LDS (a row of
// columns per slice) and from there into the matrix instruction: rows are columns, K the
// slices, columns the modes.  FP64 vector work and the FP64 matrix instruction add up
// here (at 192^3 some 65 vector instructions a voxel take 12 us and the products 6 of 31), so
// both are kept small: more slices a lane share a prefix, a full T and the addresses, and
// where a workgroup holds whole columns the products take the sums and differences of
// mirror slices against the half-axis modes, half as many.
// ---------------------------------------------------------------------------

// dV w exp(-i qc z) of a lane's K slices from z on into LDS, (Sb, Sd) the sums before the
// first, (r0, r1) the rotation there.
template <bool MSFT, int K>
__device__ __forceinline__ void ew_strength(const EwDesc& D, const float* d, const float* b, double Sb, double Sd,
                                            double r0, double r1, int z, double* re, double* im)
{
    Propagator<MSFT> P;
    P.template start<K>(Sb, Sd, b, d, D.k0dz64, r0, r1, D.step_r, D.step_i);
    const bool density = !MSFT && D.strength == MSFT_STRENGTH_DENSITY;
    auto slices = [&](auto small) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double dk = d[k], bk = b[k];
            double chr = dk * (dk - 2.0) - bk * bk, chi = 2.0 * bk * (1.0 - dk);
            if (density) {
                chr = dk;
                chi = bk;
            }
            re[slice_row(z + k)] = chr * P.tr - chi * P.ti;
            im[slice_row(z + k)] = chr * P.ti + chi * P.tr;
            if (k + 1 < K) P.template next<decltype(small)::value>(bk, dk);
        }
    };
    if (!MSFT || P.small) slices(std::true_type{});
    else slices(std::false_type{});
}

// Whole columns: COLS of them, 16 lanes of K slices each.  The products' rows are 16
// columns, Re and Im apart (COLS = 16: four waves, each one of them and one parity of the
// modes), or 8 columns' (Re, Im) (COLS = 8: two waves, a parity each).  NT tiles of 16 modes
// share an operand.  Nothing the first products need but the strength itself is waited for
// after it: their mode operands are loaded with the voxels, later ones a block of steps
// ahead.
template <bool MSFT, int COLS, int K, int NT>
__device__ __forceinline__ void ew_scan_whole(const EwReq& q, const EwDesc& D, int item, double* sm)
{
    constexpr int NZ = 16 * K, U = NT == 1 ? 8 : NT == 2 ? 6 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int cl = tid >> 4, z0 = (tid & 15) * K, nz = D.nz;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)item * COLS;
    const bool in = c0 + cl < ncol;
    const int64_t off = (in ? c0 + cl : ncol - 1) * nz;
    float d[K], b[K];
    load_slices<K>(q.delta + off, q.beta + off, z0, nz, in, d, b);
    const gcdouble rot = as_global(D.rot) + 2 * min(z0, (nz + EW_ZC - 1) / EW_ZC * EW_ZC - 1);
    const double r0 = rot[0], r1 = rot[1];
    const int odd = wave & 1, sub = wave >> 1, kze = D.kze, kz = odd ? D.kz - kze : kze, kzt = odd ? D.kzot : D.kzet;
    // whole steps of four mirror pairs; the last may be the rest (its pairs, an odd column's middle)
    const int full = nz >> 3, nh = (nz + 1) >> 1, steps = 4 * full < nh ? full + 1 : full;
    const gcdouble phi = as_global(odd ? D.phizo : D.phize);
    const uint32_t po = 8 * (lk * kzt + li);
    auto load = [&](int k, int at, double (*x)[NT]) {   // steps k ... k + U - 1, past the end the last
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const gcdouble p = phi + 4 * min(k + u, steps - 1) * kzt;
#pragma unroll
            for (int t = 0; t < NT; ++t) x[u][t] = load_at(p + (at + 16 * t < kzt ? at + 16 * t : 0), po);
        }
    };
    double x[U][NT];
    load(0, 0, x);
    __builtin_amdgcn_sched_barrier(0);
    double Sb = 0.0, Sd = 0.0;
    if (MSFT) {
        double sb = 0.0, sd = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            sb += (double)b[k];
            sd += (double)d[k];
        }
        Sb = row_prefix_f64(sb) - sb;
        Sd = row_prefix_f64(sd) - sd;
    }
    double* o = sm + (COLS == 16 ? cl : 2 * cl);
    ew_strength<MSFT, K>(D, d, b, Sb, Sd, r0, r1, z0, o, o + (COLS == 16 ? slice_row(NZ) : 1));
    __syncthreads();
    const double* a = sm + (COLS == 16 ? sub * slice_row(NZ) : 0) + li;
    const double mirror = odd ? -1.0 : 1.0;
    // slices 4 s + lk and their mirrors: eight slices on, a row offset of slice_row(8)
    const double *lo0 = a + slice_row(lk), *lo1 = a + slice_row(lk + 4);
    const double *hi0 = a + slice_row(nz - 1 - lk), *hi1 = a + slice_row(nz - 5 - lk);
    gdouble out = as_global(q.ws) + c0 * D.ld;
    const bool whole = c0 + COLS <= ncol;
    // both parities make the same passes; one past its last tile repeats the first and stores nothing
    for (int t0 = 0; t0 < max(kze, D.kz - kze); t0 += 16 * NT) {
        f64x4 t[NT];
#pragma unroll
        for (int k = 0; k < NT; ++k) t[k] = F64X4_ZERO;
        if (t0) load(0, t0, x);
        for (int k = 0; k < steps; k += U) {
            double y[U][NT];
            if (k + U < steps) load(k + U, t0, y);
            __builtin_amdgcn_sched_barrier(0);
            const int at = (k >> 1) * slice_row(8);
            if (k + U <= full) {
                double v[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int w = at + (u >> 1) * slice_row(8);
                    v[u] = (u & 1 ? hi1 : hi0)[-w] + mirror * (u & 1 ? lo1 : lo0)[w];
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < NT; ++i) t[i] = mfma_f64(v[u], x[u][i], t[i]);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (k + u < steps) {
                        const int h = min(4 * (k + u) + lk, nh - 1), m = nz - 1 - h;   // phi is zero past the middle
                        const double v = a[slice_row(m)] + (m == h ? 0.0 : mirror * a[slice_row(h)]);
#pragma unroll
                        for (int i = 0; i < NT; ++i) t[i] = mfma_f64(v, x[u][i], t[i]);
                    }
            }
            if (k + U < steps)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < NT; ++i) x[u][i] = y[u][i];
        }
#pragma unroll
        for (int k = 0; k < NT; ++k) {
            const int l = t0 + 16 * k + li;
            if (l < kz)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 4 * r + lk, col = COLS == 16 ? row : row >> 1, ri = COLS == 16 ? sub : row & 1;
                    // odd modes carry -i: (re, im) -> (im, -re)
                    if (whole || c0 + col < ncol)
                        out[col * D.ld + 2 * (odd ? kze + l : l) + (odd ? 1 - ri : ri)] =
                            odd && ri == 0 ? -t[k][r] : t[k][r];
                }
        }
    }
    // the padding of the mode vectors, zero
    const int pad = 2 * (D.kzp - D.kz);
    if ((tid & 15) < pad && in) out[cl * D.ld + 2 * D.kz + (tid & 15)] = 0.0;
}

template <typename A, bool MSFT, int COLS, int K, int NT>
__global__ __launch_bounds__(16 * COLS, K == 16 ? 2 : NT > 1 || COLS == 8 ? 3 : 4) void ew_scan_kernel(A args)
{
    __shared__ double sm[(COLS == 16 ? 2 : 1) * slice_row(16 * K)];   // Re and Im; or (Re, Im) rows
    int item;
    const EwReq& q = ew_request(args, item);
    ew_scan_whole<MSFT, COLS, K, NT>(q, ew_desc(args, q), item, sm);
}

// Longer columns, in rounds of 64 slices against the full-axis modes.  Wave w takes Re (w
// even) or Im of mode tiles w / 2, w / 2 + 2, ...
template <typename A, bool MSFT>
__global__ __launch_bounds__(EW_THREADS) void ew_scan_rounds_kernel(A args)
{
    constexpr int NT = EW_MAX_KZ / 32;
    __shared__ double sm[2 * slice_row(EW_ZC)];
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int cl = tid >> 4, zl = (tid & 15) * 4, nz = D.nz, kzt = D.kzt;
    const int64_t ncol = (int64_t)D.nx * D.ny, c0 = (int64_t)item * EW_COLS;
    const bool in = c0 + cl < ncol;
    const int64_t off = (in ? c0 + cl : ncol - 1) * nz;
    const int ri = wave & 1, t0 = wave >> 1;
    const gcdouble phi = as_global(D.phiz) + t0 * 16, rot = as_global(D.rot) + 2 * zl;
    const uint32_t po = 8 * (lk * kzt + li);
    f64x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = F64X4_ZERO;
    double carry_b = 0.0, carry_d = 0.0;
    float d[4], b[4];
    for (int z0 = 0; z0 < nz; z0 += EW_ZC) {
        load_slices<4>(q.delta + off, q.beta + off, z0 + zl, nz, in, d, b);
        double Sb = 0.0, Sd = 0.0;
        if (MSFT) {
            const double sb = ((double)b[0] + b[1]) + ((double)b[2] + b[3]);
            const double sd = ((double)d[0] + d[1]) + ((double)d[2] + d[3]);
            const double ib = row_prefix_f64(sb), id = row_prefix_f64(sd);
            Sb = carry_b + (ib - sb);
            Sd = carry_d + (id - sd);
            carry_b += row_last_f64(ib);
            carry_d += row_last_f64(id);
        }
        ew_strength<MSFT, 4>(D, d, b, Sb, Sd, rot[2 * z0], rot[2 * z0 + 1], zl, sm + cl, sm + slice_row(EW_ZC) + cl);
        __syncthreads();
        const double* a = sm + ri * slice_row(EW_ZC) + li;
        for_steps<4>(EW_ZC / 4, [&](int ks) {
            const double v = a[slice_row(4 * ks + lk)];
            const gcdouble p = phi + (int64_t)(z0 + 4 * ks) * kzt;
#pragma unroll
            for (int t = 0; t < NT; ++t)   // a wave past the last tile repeats the first and stores nothing
                acc[t] = mfma_f64(v, load_at(p + ((t0 + 2 * t) * 16 < kzt ? 32 * t : -16 * t0), po), acc[t]);
        });
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int l = (t0 + 2 * t) * 16 + li;
        if (l >= D.kzp) continue;
        const bool odd = l >= D.kze;   // -i: (re, im) -> (im, -re)
        const int comp = odd ? 1 - ri : ri;
        const double sign = odd && ri == 0 ? -1.0 : 1.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t col = c0 + 4 * r + lk;
            if (col < ncol) q.ws[col * D.ld + 2 * l + comp] = sign * acc[t][r];
        }
    }
}

// ---------------------------------------------------------------------------
// Sums over half an axis: t[0], t[1] += te (v[hi] + v[lo]), t[2], t[3] += to (v[hi] - v[lo])
// for voxels hi = n - 1 - h, lo = h, rows of `stride` doubles at v, the lane's column at
// byte 8 cc; te, to tables of `ldE`, `ldO` doubles a row, two tiles each.  The waves of
// the workgroup take every fourth step of four pairs; the last step (its pairs, an odd
// axis's middle voxel; the tables are zero past it) is one wave's.  The addresses of
// whole steps are scalar.  Two steps' loads are issued ahead: four take 144 registers
// instead of 73, and the waves lost cost more (256^3/1024^2: modal 77 us instead of 64,
// nodes 103 instead of 88; eight mixed requests 23.4 and 20.1 instead of 18.5 and 16.2).
// ---------------------------------------------------------------------------
struct HalfAxis {
    gcdouble v, e0, e1, o0, o1;
    int64_t stride;
    int n, ldE, ldO, cc;
};

__device__ __forceinline__ void half_axis_sums(const HalfAxis& x, int wave, int li, int lk, f64x4* t)
{
    const int full = x.n >> 3, nh = (x.n + 1) >> 1, h0 = 4 * wave;
    const uint32_t pe = 8 * (lk * x.ldE + li), po = 8 * (lk * x.ldO + li);
    const int64_t v16 = 16 * x.stride, e16 = 16 * x.ldE, o16 = 16 * x.ldO;
    const Stream s[6] = {{x.v + (x.n - 4 - h0) * x.stride, -v16, 8 * (uint32_t)((3 - lk) * x.stride + x.cc)},
                         {x.v + h0 * x.stride, v16, 8 * (uint32_t)(lk * x.stride + x.cc)},
                         {x.e0 + h0 * x.ldE, e16, pe},
                         {x.e1 + h0 * x.ldE, e16, pe},
                         {x.o0 + h0 * x.ldO, o16, po},
                         {x.o1 + h0 * x.ldO, o16, po}};
    staged<2>(s, (full - wave + 3) >> 2, [&](int, const double* y) {
        const double sum = y[0] + y[1], diff = y[0] - y[1];
        t[0] = mfma_f64(y[2], sum, t[0]);
        t[1] = mfma_f64(y[3], sum, t[1]);
        t[2] = mfma_f64(y[4], diff, t[2]);
        t[3] = mfma_f64(y[5], diff, t[3]);
    });
    if (4 * full < nh && wave == (full & 3)) {
        const int h = min(4 * full + lk, nh - 1), hi = x.n - 1 - h;
        const double vh = x.v[hi * x.stride + x.cc], vl = hi == h ? 0.0 : x.v[h * x.stride + x.cc];
        t[0] = mfma_f64(load_at(x.e0 + 4 * full * x.ldE, pe), vh + vl, t[0]);
        t[1] = mfma_f64(load_at(x.e1 + 4 * full * x.ldE, pe), vh + vl, t[1]);
        t[2] = mfma_f64(load_at(x.o0 + 4 * full * x.ldO, po), vh - vl, t[2]);
        t[3] = mfma_f64(load_at(x.o1 + 4 * full * x.ldO, po), vh - vl, t[3]);
    }
}

// ---------------------------------------------------------------------------
// Modal: Y[N][m][c] = sum_h phi_m(h) (Z[hi] +- Z[lo])[c], c the 2 kzp doubles of a mode
// vector.  A workgroup takes one N, 16 values of c and two tiles of 16 modes of each
// parity: a pair of loads feeds four products.  The groups of modes of one (N, c) follow
// each other on one XCD (workgroups go to the eight XCDs in turn), so that its L2 holds
// their Z after the first.
// ---------------------------------------------------------------------------
template <typename A>
__global__ __launch_bounds__(EW_THREADS) void ew_modal_kernel(A args)
{
    __shared__ double red[SUM_WAVES_LDS];
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, ct = (ld + 15) >> 4, groups = (max(D.ket, D.kop ? D.kot : 0) + 31) >> 5;
    const int g = (item >> 3) % groups, u = (item >> 3) / groups * 8 + (item & 7);
    const int N = u / ct, c = u % ct * 16 + li;
    if (N >= D.nN) return;   // workgroup-uniform
    const int ket = D.ket, kot = D.kot;
    // tiles past a parity's last repeat its first; their rows are not stored
    HalfAxis x;
    x.v = as_global(q.ws) + (int64_t)N * D.zsN * ld;
    x.stride = (int64_t)D.zsM * ld;
    x.n = D.nM;
    x.cc = min(c, ld - 1);
    x.ldE = ket;
    x.ldO = kot;
    x.e0 = as_global(D.phie) + (g * 32 < ket ? g * 32 : 0);
    x.e1 = as_global(D.phie) + (g * 32 + 16 < ket ? g * 32 + 16 : 0);
    x.o0 = as_global(D.phio) + (g * 32 < kot ? g * 32 : 0);
    x.o1 = as_global(D.phio) + (g * 32 + 16 < kot ? g * 32 + 16 : 0);
    f64x4 t[4] = {F64X4_ZERO, F64X4_ZERO, F64X4_ZERO, F64X4_ZERO};
    half_axis_sums(x, wave, li, lk, t);
    const f64x4 s = sum_waves(red, t, wave, lane);
    const bool odd = wave >= 2;
    const int m0 = g * 32 + 16 * (wave & 1), kp = odd ? D.kop : D.kep;
    gdouble y = as_global(q.ws) + D.offY + ((int64_t)N * D.km + (odd ? D.kep : 0) + m0) * ld;
    if (c < ld)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (m0 + 4 * r + lk < kp) y[(4 * r + lk) * ld + c] = s[r];
}

// ---------------------------------------------------------------------------
// Nodes: G[a][cos|sin][m][c] = sum_h {cos, sin}(q_N(a) N_h) (Y[hi] +- Y[lo])[m][c].  A
// workgroup takes 16 of the km * 2 kzp columns and two tiles of 16 values of a, both
// parities; the groups of a of one column tile on one XCD.
// ---------------------------------------------------------------------------
template <typename A>
__global__ __launch_bounds__(EW_THREADS) void ew_nodes_kernel(A args)
{
    __shared__ double red[SUM_WAVES_LDS];
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ncols = D.km * D.ld, nap = D.nap, ga = (min(nap - q.a0, D.chunk) + 31) >> 5;
    const int g = (item >> 3) % ga, cb = ((item >> 3) / ga * 8 + (item & 7)) * 16;
    if (cb >= ncols) return;   // workgroup-uniform
    const int a0 = q.a0 + g * 32, a1 = a0 + 16 < nap ? a0 + 16 : a0, c = cb + li;
    HalfAxis x;
    x.v = as_global(q.ws) + D.offY;
    x.stride = ncols;
    x.n = D.nN;
    x.cc = min(c, ncols - 1);
    x.ldE = x.ldO = nap;
    x.e0 = as_global(D.cosN) + a0;
    x.e1 = as_global(D.cosN) + a1;
    x.o0 = as_global(D.sinN) + a0;
    x.o1 = as_global(D.sinN) + a1;
    f64x4 t[4] = {F64X4_ZERO, F64X4_ZERO, F64X4_ZERO, F64X4_ZERO};
    half_axis_sums(x, wave, li, lk, t);
    const f64x4 s = sum_waves(red, t, wave, lane);
    const int first = a0 + 16 * (wave & 1);
    gdouble out = as_global(q.ws) + D.offG + (2 * (first - q.a0) + (wave >> 1)) * (int64_t)ncols;
    if (c < ncols && first < nap)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (first + 4 * r + lk < D.na) out[(int64_t)(2 * (4 * r + lk)) * ncols + c] = s[r];
}

// ---------------------------------------------------------------------------
// yz: S[pN][pM](a, b) = sum_l c_l(a, b) sum_{m in pM} c_m(a, b) G[a][pN][m][l].  A
// workgroup takes one a and BT tiles of 16 b (the rows); a wave one pM and every other
// tile of 16 columns (l, re | im), K running over the modes m, both pN sharing the c_m
// operand and the BT tiles the G operand.  c_l multiplies each product tile, and the
// columns are summed at the end over lanes and waves.  With one tile three steps' loads are
// issued ahead (more waves: 26.5 us against 31 with six at 132^3, 13.5 nm), with two, which
// read G half as often, six (256^3/1024^2: 142 us, three 151; one tile 166).  The result goes to
// [4 px + 2 py + (re | im)][row node][node], px and py the parities along x and y.  The
// groups of b of one a follow each other on one XCD.
// ---------------------------------------------------------------------------
template <typename A, int BT>
__global__ __launch_bounds__(EW_THREADS) void ew_yz_kernel(A args)
{
    __shared__ double red[2][2][2][BT * 16][2];   // [column half][pM][pN][b][ri]
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int ld = D.ld, nbp = D.nbp, kzp = D.kzp, bg = (nbp + 16 * BT - 1) / (16 * BT);
    const int al = (item >> 3) / bg * 8 + (item & 7), a = q.a0 + al, b0 = (item >> 3) % bg * (16 * BT);
    if (al >= D.chunk || a >= D.na) return;   // workgroup-uniform
    const int pm = wave & 1, half = wave >> 1;
    const int m0 = pm ? D.kep : 0, steps = (pm ? D.kop : D.kep) >> 2;
    const int64_t gs = (int64_t)D.km * ld;
    const gcdouble gm = as_global(q.ws) + D.offG + 2 * al * gs + (int64_t)m0 * ld;
    const gcdouble cm = as_global(D.cm) + ((int64_t)a * D.km + m0) * nbp;
    const gcdouble cz = as_global(D.cz) + (int64_t)a * nbp * kzp;
    const uint32_t om = 8 * (lk * nbp + li);
    int bt[BT];   // a tile past the last repeats it
#pragma unroll
    for (int k = 0; k < BT; ++k) bt[k] = min(b0 + 16 * k, nbp - 16);
    double s[2][BT][4];
#pragma unroll
    for (int k = 0; k < BT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) s[0][k][r] = s[1][k][r] = 0.0;
    for (int c0 = 16 * half; c0 < ld; c0 += 32) {
        const int c = c0 + li, x = min(c, ld - 1);
        const uint32_t og = 8 * (lk * ld + x), oz = 8 * (lk * kzp + (x >> 1));
        double z[BT][4];
#pragma unroll
        for (int k = 0; k < BT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                z[k][r] = load_at(cz + (bt[k] + 4 * r) * kzp, oz);
                if (c >= ld) z[k][r] = 0.0;
            }
        f64x4 e[BT], o[BT];
#pragma unroll
        for (int k = 0; k < BT; ++k) e[k] = o[k] = F64X4_ZERO;
        Stream g[2 + BT];
        g[0] = {gm, 4 * ld, og};
        g[1] = {gm + gs, 4 * ld, og};
#pragma unroll
        for (int k = 0; k < BT; ++k) g[2 + k] = {cm + bt[k], 4 * nbp, om};
        staged<BT == 2 ? 6 : 3>(g, steps, [&](int, const double* y) {
#pragma unroll
            for (int k = 0; k < BT; ++k) {
                e[k] = mfma_f64(y[2 + k], y[0], e[k]);
                o[k] = mfma_f64(y[2 + k], y[1], o[k]);
            }
        });
#pragma unroll
        for (int k = 0; k < BT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[0][k][r] += e[k][r] * z[k][r];
                s[1][k][r] += o[k][r] * z[k][r];
            }
    }
    // sum the lanes of one row with the same re | im (lane bits 1 - 3)
#pragma unroll
    for (int k = 0; k < BT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                double v = s[p][k][r];
                v += dpp_f64<0x4E, 0xF>(v);    // quad_perm 2,3,0,1
                v += dpp_f64<0x124, 0xF>(v);   // row_ror 4
                v += dpp_f64<0x128, 0xF>(v);   // row_ror 8
                if (li < 2) red[half][pm][p][16 * k + 4 * r + lk][li] = v;
            }
    __syncthreads();
    const int uni = D.uniform;
    for (int t = threadIdx.x; t < BT * 16 * 8; t += EW_THREADS) {
        const int comp = t / (BT * 16), bl = t % (BT * 16), b = b0 + bl;
        if (b >= D.nb) continue;
        const int px = comp >> 2, py = (comp >> 1) & 1, pn = uni ? py : px, p = uni ? px : py;
        const double v = red[0][p][pn][bl][comp & 1] + red[1][p][pn][bl][comp & 1];
        const int row = uni ? a : b, node = uni ? b : a;
        q.ws[D.offS + ((int64_t)comp * D.nr + row) * D.n + node] = v;
    }
}

// ---------------------------------------------------------------------------
// Coef: C[row][k][comp] = sum_a D[a][k] sum_r W[row][r] S[comp][r][a] for 16 pixel rows and
// one of the eight parts: two products on the matrix instruction, the first one's result
// through LDS (a row of 16 per node, padded to 17), a wave to a tile of 16 nodes and then
// of 16 coefficients.  W by the part's parity in the rows' angle (along y), D by its
// parity in the pixels' (along x).  The eight parts of a row follow each other on one
// XCD, whose L2 merges their pieces of C.
// ---------------------------------------------------------------------------
constexpr int CF_THREADS = 1024;   // at most: a wave to every 16 nodes

template <typename A>
__global__ __launch_bounds__(CF_THREADS) void ew_coef_kernel(A args)
{
    extern __shared__ double lds[];   // [n][17]
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int lane = threadIdx.x & 63, wave = wave_index(), li = lane & 15, lk = lane >> 4;
    const int n = D.n, nr = D.nr, rowsp = D.rowsp, np = (n + 15) & ~15, waves = blockDim.x >> 6;
    const int comp = (item >> 3) & 7, j0 = ((item >> 6) * 8 + (item & 7)) * 16;
    if (j0 >= D.rows) return;
    const int px = comp >> 2, py = (comp >> 1) & 1;
    {
        const gcdouble w = as_global(py ? D.wro : D.wre) + j0, s = as_global(q.ws) + D.offS + (int64_t)comp * nr * n;
        const uint32_t ow = 8 * (lk * rowsp + li);
        for (int a0 = 16 * wave; a0 < n; a0 += 16 * waves) {
            const int a = min(a0 + li, n - 1);
            const uint32_t os = 8 * (lk * n + a);
            f64x4 t = F64X4_ZERO;
            const Stream x[2] = {{w, 4 * rowsp, ow}, {s, 4 * n, os}};
            staged<8>(x, nr >> 2, [&](int, const double* y) { t = mfma_f64(y[0], y[1], t); });
            if (nr & 3) {   // W is zero past nr
                const int r = nr & ~3;
                t = mfma_f64(load_at(w + r * rowsp, ow), s[min(r + lk, nr - 1) * n + a], t);
            }
            if (a0 + li < n)
#pragma unroll
                for (int r = 0; r < 4; ++r) lds[(a0 + li) * 17 + 4 * r + lk] = t[r];
        }
    }
    __syncthreads();
    const gcdouble m = as_global(px ? D.dcto : D.dcte);
    const uint32_t om = 8 * (lk * np + li);
    gdouble out = as_global(q.ws) + D.offC + comp;
    for (int k0 = 16 * wave; k0 < n; k0 += 16 * waves) {
        f64x4 t = F64X4_ZERO;
        const Stream x[1] = {{m + k0, 4 * np, om}};
        staged<8>(x, n >> 2, [&](int ks, const double* y) { t = mfma_f64(lds[(4 * ks + lk) * 17 + li], y[0], t); });
        if (n & 3) {   // D is zero past n
            const int a = n & ~3;
            t = mfma_f64(lds[min(a + lk, n - 1) * 17 + li], load_at(m + a * np + k0, om), t);
        }
        const int k = k0 + li;
        if (k < n)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + 4 * r + lk;
                if (j < D.rows) out[((int64_t)j * n + k) * 8] = t[r];
            }
    }
}

// ---------------------------------------------------------------------------
// Eval: a workgroup takes up to 128 CPL columns of one pixel row, the row's coefficients in
// LDS.  Of each pair of waves one runs the recurrence of T_2k in x = 2 t^2 - 1 with the four
// parts even along the row, the other that of T_2k+1 with the odd ones, for CPL columns a
// lane.  It is bound by the vector unit and by LDS, whose broadcast of a coefficient takes
// as long as four products: at CPL = 4 as at 2 a lane's columns share it, at 4 enough that
// the vector unit is the longer of the two.  The parts' sums meet in the even wave,
//   A(sx, sy) = (ee - sx sy oo) - i (sx oe + sy eo)          (px, py)
// for the four mirror pixels.  One wave for both series, two columns a lane, took 8.0 us at
// 128^3/512^2 and 43.7 at 256^3/1024^2, against 5.4 and 32.8.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void ew_store(const EwReq& q, int N, int i, int j, bool rim, const double* s)
{
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const bool px = !(m & 1), py = !(m & 2);   // the pixel at +u, +v
        const int ii = px ? N - 1 - i : i, jj = py ? N - 1 - j : j;
        if ((!px && ii == N - 1 - i) || (!py && jj == N - 1 - j)) continue;   // the middle, done at +
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

constexpr int EV_THREADS = 256;   // at most: two pairs of waves

template <typename A, int CPL>
__global__ __launch_bounds__(EV_THREADS) void ew_eval_kernel(A args)
{
    extern __shared__ double C[];   // [n][8], then the odd sums [pair][column][4][64]
    int item;
    const EwReq& q = ew_request(args, item);
    const EwDesc& D = ew_desc(args, q);
    const int n = D.n, N = D.det_n, half = D.rows, tid = threadIdx.x, lane = tid & 63, wave = wave_index();
    const int cols = blockDim.x / 2 * CPL, chunks = (half + cols - 1) / cols, j = item / chunks;
    // nothing to do where the row and its mirror lie outside [p0, p1)
    const int64_t lo = (int64_t)j * N, hi = (int64_t)(N - 1 - j) * N;
    if ((lo + N <= q.p0 || lo >= q.p1) && (hi + N <= q.p0 || hi >= q.p1)) return;
    const gcdouble tq = as_global(D.tq) + (int64_t)j * half;
    const int odd = wave & 1, pair = wave >> 1, i = item % chunks * cols + pair * (64 * CPL) + lane;
    double f0[CPL], f1[CPL], x2[CPL], s[CPL][8];
#pragma unroll
    for (int p = 0; p < CPL; ++p) f0[p] = tq[min(i + 64 * p, half - 1)];
    const double2* src = (const double2*)(q.ws + D.offC + (int64_t)j * n * 8);
    for (int k = tid; k < n * 4; k += blockDim.x) ((double2*)C)[k] = src[k];
    uint32_t rim = 0;
#pragma unroll
    for (int p = 0; p < CPL; ++p) {
        if (!(f0[p] == f0[p])) {
            rim |= 1u << p;
            f0[p] = 0.0;
        }
        const double t = f0[p];
        x2[p] = 2.0 * (2.0 * t * t - 1.0);
        f0[p] = odd ? t : 1.0;                              // T_1 or T_0
        f1[p] = odd ? (x2[p] - 1.0) * t : 0.5 * x2[p];      // T_3 or T_2
#pragma unroll
        for (int c = 0; c < 4; ++c) s[p][c] = 0.0;
    }
    __syncthreads();
    const double* c4 = C + 4 * odd;
#pragma unroll 4
    for (int k = 0; k < n; ++k)
#pragma unroll
        for (int p = 0; p < CPL; ++p) {
#pragma unroll
            for (int c = 0; c < 4; ++c) s[p][c] += f0[p] * c4[k * 8 + c];
            const double f2 = x2[p] * f1[p] - f0[p];
            f0[p] = f1[p];
            f1[p] = f2;
        }
    double* sums = C + n * 8 + pair * (CPL * 4 * 64) + lane;
    if (odd)
#pragma unroll
        for (int k = 0; k < CPL * 4; ++k) sums[k * 64] = s[k >> 2][k & 3];
    __syncthreads();
    if (odd) return;
#pragma unroll
    for (int p = 0; p < CPL; ++p) {
        if (i + 64 * p >= half) break;
#pragma unroll
        for (int c = 0; c < 4; ++c) s[p][4 + c] = sums[(p * 4 + c) * 64];
        ew_store(q, N, i + 64 * p, j, rim >> p & 1, s[p]);
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

// The other angle of pixel (row j, column i) over its range, the Chebyshev argument of the
// row's series; NaN beyond the rim, by the q map's own comparison (no contraction).
__global__ void ew_argument_kernel(EwDesc D, double k0, double limit, double scale, double* tq)
{
#pragma clang fp contract(off)
    const int half = D.rows;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int j = (int)(t / half), i = (int)(t % half);
    if (j >= half) return;
    const double u = ((double)(D.det_n - 1 - 2 * i) * limit) / (double)D.det_n;
    const double v = ((double)(D.det_n - 1 - 2 * j) * limit) / (double)D.det_n;
    const double s = u * u + v * v, kk = k0 * k0;
    double w;
    if (!D.uniform) w = atan(u * cos(atan(v)));
    else w = s < kk ? atan2(u, sqrt(kk - s)) : __builtin_nan("");
    tq[t] = w * scale;
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
__global__ __launch_bounds__(256) void ew_mode_kernel(CoefArgs c)
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

EwReq ew_one(const EwReq& r, const EwDesc&, EwReq*) { return r; }
EwOne ew_one(const EwReq& r, const EwDesc& d, EwOne*) { return {r, d}; }

// One launch over all requests, f(plan) workgroups to each.
template <typename A, typename F>
void ew_launch(void (*one)(A), void (*many)(EwBatch), EwBatch& b, const EwDesc* const* dims, int lds,
               hipStream_t s, F f, int threads = EW_THREADS)
{
    if (b.n == 1) {
        hipLaunchKernelGGL(one, dim3((unsigned)f(*dims[0])), dim3(threads), lds, s, ew_one(b.req[0], *dims[0], (A*)nullptr));
        return;
    }
    int64_t total = 0;
    for (int r = 0; r < b.n; ++r) {
        b.begin[r] = (int32_t)total;
        total += f(*dims[r]);
    }
    b.begin[b.n] = (int32_t)total;
    hipLaunchKernelGGL(many, dim3((unsigned)total), dim3(threads), lds, s, b);
}

// Workgroups of a kernel whose `inner` workgroups of each of `outer` units follow each
// other on one XCD.
int64_t ew_on_xcd(int64_t outer, int64_t inner) { return ceil_div(outer, 8) * 8 * inner; }

// The scan's form for a plan: its rounding goes by its own columns in any batch.
struct ScanForm {
    int rounds, tiles;
    bool msft;
    explicit ScanForm(const EwDesc& d)
        : rounds(ew_rounds(d.nz)), tiles(rounds ? std::min(3, std::max(d.kzet, d.kzot) / 16) : 0),
          msft(d.strength == MSFT_STRENGTH_MSFT)
    {
    }
    bool operator==(const ScanForm& o) const { return rounds == o.rounds && tiles == o.tiles && msft == o.msft; }
};

template <bool MSFT, int COLS, int K>
void ew_launch_scan(EwBatch& b, const EwDesc* const* dims, int tiles, hipStream_t s)
{
    auto items = [](const EwDesc& d) { return ceil_div((int64_t)d.nx * d.ny, COLS); };
    if (tiles == 1) ew_launch(ew_scan_kernel<EwOne, MSFT, COLS, K, 1>, ew_scan_kernel<EwBatch, MSFT, COLS, K, 1>, b, dims, 0, s, items, 16 * COLS);
    else if (tiles == 2) ew_launch(ew_scan_kernel<EwOne, MSFT, COLS, K, 2>, ew_scan_kernel<EwBatch, MSFT, COLS, K, 2>, b, dims, 0, s, items, 16 * COLS);
    else ew_launch(ew_scan_kernel<EwOne, MSFT, COLS, K, 3>, ew_scan_kernel<EwBatch, MSFT, COLS, K, 3>, b, dims, 0, s, items, 16 * COLS);
}

template <bool MSFT>
void ew_launch_scan(EwBatch& b, const EwDesc* const* dims, const ScanForm& f, hipStream_t s)
{
    switch (f.rounds) {
    case 1: ew_launch_scan<MSFT, 16, 4>(b, dims, f.tiles, s); break;
    case 2: ew_launch_scan<MSFT, 16, 8>(b, dims, f.tiles, s); break;
    case 3: ew_launch_scan<MSFT, 8, 12>(b, dims, f.tiles, s); break;
    case 4: ew_launch_scan<MSFT, 8, 16>(b, dims, f.tiles, s); break;
    default:
        ew_launch(ew_scan_rounds_kernel<EwOne, MSFT>, ew_scan_rounds_kernel<EwBatch, MSFT>, b, dims, 0, s,
                  [](const EwDesc& d) { return ceil_div((int64_t)d.nx * d.ny, EW_COLS); });
    }
}

}  // namespace

int launch_ew_scan(const EwBatch& b, const EwDesc* const* dims, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    bool done[EW_MAX_REQ] = {};
    for (int first = 0; first < b.n; ++first) {   // the requests of one form together
        if (done[first]) continue;
        const ScanForm form(*dims[first]);
        EwBatch part;
        const EwDesc* d[EW_MAX_REQ];
        part.n = 0;
        for (int r = first; r < b.n; ++r)
            if (!done[r] && ScanForm(*dims[r]) == form) {
                done[r] = true;
                d[part.n] = dims[r];
                part.req[part.n++] = b.req[r];
            }
        if (form.msft) ew_launch_scan<true>(part, d, form, s);
        else ew_launch_scan<false>(part, d, form, s);
    }
    return (int)hipGetLastError();
}

int launch_ew_contract(EwBatch& b, const EwDesc* const* dims, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    int n = 0;
    for (int r = 0; r < b.n; ++r) n = std::max(n, dims[r]->n);
    ew_launch(ew_modal_kernel<EwReq>, ew_modal_kernel<EwBatch>, b, dims, 0, s, [](const EwDesc& d) {
        return ew_on_xcd(d.nN * ceil_div(d.ld, 16), ceil_div(std::max(d.ket, d.kop ? d.kot : 0), 32));
    });
    // G in parts where a request's workspace holds fewer nodes than all: part k of each request
    for (int k = 0;; ++k) {
        EwBatch part;
        const EwDesc* d[EW_MAX_REQ];
        int64_t bt = 0;
        part.n = 0;
        for (int r = 0; r < b.n; ++r) {
            const int a0 = k * dims[r]->chunk;
            if (a0 >= dims[r]->na) continue;
            bt += (int64_t)std::min(dims[r]->chunk, dims[r]->na - a0) * (dims[r]->nbp / 16);
            d[part.n] = dims[r];
            part.req[part.n] = b.req[r];
            part.req[part.n++].a0 = a0;
        }
        if (part.n == 0) break;
        ew_launch(ew_nodes_kernel<EwReq>, ew_nodes_kernel<EwBatch>, part, d, 0, s, [&](const EwDesc& e) {
            return ew_on_xcd(ceil_div((int64_t)e.km * e.ld, 16), ceil_div(std::min(e.nap - k * e.chunk, e.chunk), 32));
        });
        auto tiles = [&](const EwDesc& e, int b16) {
            return ew_on_xcd(std::min(e.na - k * e.chunk, e.chunk), ceil_div(e.nbp, 16 * b16));
        };
        if (bt >= 8 * CHIP_CUS)
            ew_launch(ew_yz_kernel<EwReq, 2>, ew_yz_kernel<EwBatch, 2>, part, d, 0, s, [&](const EwDesc& e) { return tiles(e, 2); });
        else
            ew_launch(ew_yz_kernel<EwReq, 1>, ew_yz_kernel<EwBatch, 1>, part, d, 0, s, [&](const EwDesc& e) { return tiles(e, 1); });
    }
    ew_launch(ew_coef_kernel<EwReq>, ew_coef_kernel<EwBatch>, b, dims, n * 17 * (int)sizeof(double), s,
              [](const EwDesc& d) { return ew_on_xcd(d.rowsp / 16, 8); },
              std::min(CF_THREADS, std::max(4, (n + 15) / 16) * 64));
    // four columns a lane where that leaves two waves to a SIMD and the series are long
    // (512^2 quarter pixels, 235 coefficients: 33 us against 39; 57: 12.7 against 13.2, eight
    // mixed requests of 57: 18.6 against 18.1), else two; a pair of waves only for what a row has
    int64_t waves = 0;
    int rows = 0;
    for (int r = 0; r < b.n; ++r) {
        waves += 2 * dims[r]->rows * ceil_div(dims[r]->rows, 256);
        rows = std::max(rows, dims[r]->rows);
    }
    const int cpl = waves >= 8 * CHIP_CUS && n >= 128 ? 4 : 2, pairs = rows > 64 * cpl ? 2 : 1;
    const int lds = (n * 8 + pairs * cpl * 4 * 64) * (int)sizeof(double);
    auto items = [&](const EwDesc& d) { return d.rows * ceil_div(d.rows, pairs * 64 * cpl); };
    if (cpl == 4) ew_launch(ew_eval_kernel<EwReq, 4>, ew_eval_kernel<EwBatch, 4>, b, dims, lds, s, items, pairs * 128);
    else ew_launch(ew_eval_kernel<EwReq, 2>, ew_eval_kernel<EwBatch, 2>, b, dims, lds, s, items, pairs * 128);
    return (int)hipGetLastError();
}

int launch_ew_tables(const EwHost& h, const EwDesc& D, const EwTables& t, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(ew_trig_kernel, dim3((unsigned)ceil_div((int64_t)D.nhNp * D.nap, 256)), dim3(256), 0, s,
                       D, t.ang_a, h.k0, h.pitchN, t.cosN, t.sinN);
    hipLaunchKernelGGL(ew_argument_kernel, dim3((unsigned)ceil_div((int64_t)D.rows * D.rows, 256)), dim3(256), 0, s,
                       D, h.k0, h.limit, h.range > 0.0 ? 1.0 / h.range : 0.0, t.tq);
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
    hipLaunchKernelGGL(ew_mode_kernel, grid, dim3(256), 0, s, c);
    c.even = D.phize;
    c.odd = D.phizo;
    c.ldE = D.kzet;
    c.ldO = D.kzot;
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
    hipLaunchKernelGGL(ew_mode_kernel, grid, dim3(256), 0, s, c);
    return (int)hipGetLastError();
}

}  // namespace msft
