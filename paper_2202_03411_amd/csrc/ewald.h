// The forward model and its adjoint in spherical coordinates about a detector axis
// (internal; shared by the host plan code and the gfx950 kernels).
//
// Every pixel of either detector looks at a point of the Ewald sphere,
//   q + k0 zhat = k0 (sin a, cos a sin b, cos a cos b)   along (N, M, z),
// so q_N depends on a alone.  The flat detector takes N = x, M = y: tan b = v, so a
// pixel row j is one value of b, and tan a = u cos b.  The uniform-q detector takes
// N = y, M = x: a pixel row j is one value of a (sin a = q_y / k0).  Either way one
// angle belongs to the row and the other to the pixel, and A is an entire function of
// both: its Chebyshev series over the detector's range end, to rounding, after about
// k0 |r|_max range terms, however many pixels there are.  So
//   scan    Z_l(x, y)   = sum_z phi_l(z) exp(-i qc z) w            (modes l of q_z)
//   modal   Y_ml(N)     = sum_M phi_m(M) Z_l                       (modes m of q_M)
//   nodes   G_ml(a)     = sum_N {cos, sin}(q_N(a) N) Y_ml          (per node a)
//   yz      S(a, b)     = sum_m c_m(q_M) sum_l c_l(q_z) G_ml(a)    (per pair of nodes)
//   coef    C(row, k)   = S interpolated to the rows' angle, its Chebyshev
//                         coefficients k in the other
//   eval    A(pixel)    = sum_k T_k(t) C(row, k)
// in FP64 throughout, w included.  phi are the discrete prolate
// sequences of each axis's momentum range: the smallest basis that holds exp(-i q r)
// of every q in the range on the axis's voxel centres.  They are even or odd, as are
// cos and sin, so the sums run over half an axis of folded values, and the four
// even/odd parts of S give the four mirror pixels (+-u, +-v) at once.
#pragma once

#include <cstdint>
#include <vector>

#include "msft.h"

namespace msft {

// Least pixels x voxels a plan asks for the form with (which direction then takes it: forms.cpp).
// The form's six launches take 19 us of the host each way, the direct
// form's two or three 6 to 9.  Flat, a pattern and a gradient: 16^3 voxels on 64^2 pixels
// (1.7e7) 23 and 162 us against 33 and 145, 32^3 on 64^2 (1.3e8) 24 and 163 against 70 and
// 171.  Uniform: 32^3 on 128^2 (5.4e8) 26 and 161 against 23 and 150, 64^3 on 64^2 (1.1e9) 30
// and 163 against 35 and 177, on 256^2 32 and 161 against 47 and 177.
constexpr double EW_MIN_TERMS = 2e7;
constexpr double EW_MIN_TERMS_UNIFORM = 8e8;
constexpr int EW_COLS = 16;       // columns (x, y) of one scan workgroup: the MFMA rows
constexpr int EW_ZC = 64;         // slices of one scan round: a column's 16 lanes, four each
// Columns of at most 256 slices are held whole: 16 columns of 16 lanes up to 128 slices (4 or
// 8 a lane), beyond that 8 columns, in the scan 16 lanes of 12 or 16 slices each (32 lanes of
// 6, whose prefixes and addresses weigh twice as much, took 36.7 us at 192^3 against 30.8),
// in the adjoint's walk, which holds more registers a slice, 32 lanes of 6 or 8.  The
// strengths take at most 35 KB of LDS.
constexpr int EW_WHOLE_NZ = 256;
inline int ew_rounds(int nz) { return nz > EW_WHOLE_NZ ? 0 : (nz + EW_ZC - 1) / EW_ZC; }
inline int ew_columns(int nz) { return nz > 2 * EW_ZC && nz <= EW_WHOLE_NZ ? 8 : EW_COLS; }
constexpr int EW_MAX_KZ = 256;    // most modes of z: a scan wave keeps them in registers
constexpr int EW_MAX_KM = 1024;   // most modes of the M axis
constexpr int EW_MAX_NODES = 400; // most Chebyshev nodes: 17 doubles of LDS each, 54 KB (the adjoint: 79 KB)
constexpr int EW_LDS = 160 * 1024;   // of one workgroup, at most all of a compute unit's

// One plan's sizes and resident tables, as the kernels see them (device memory).
// Modes are ordered even, then odd; counts ending in p are padded (tables hold zeros there).
struct EwDesc {
    int32_t nx, ny, nz, strength;
    double k0dz64, dV64;
    int32_t uniform;            // N = y and M = x (else N = x, M = y)
    int32_t nN, nM, nhN, nhM;   // voxels along N and M, and half of them rounded up
    int32_t zsN, zsM;           // column strides of N and M in Z (columns x * ny + y)
    int32_t kze, kz, kzp, kzt;  // even z modes, all, padded to 4, padded to 16
    int32_t kzet, kzot;         // row lengths of phize, phizo (padded to 16)
    int32_t kep, kop, km;       // M modes: even and odd padded to 4, their sum
    int32_t ket, kot;           // row lengths of phi_e, phi_o (padded to 16)
    int32_t ld;                 // 2 kzp: doubles of one complex mode vector
    int32_t na, nap, nb, nbp;   // nodes a and b, padded to 16
    int32_t nhNp, nhMp;         // half axes padded to 16
    int32_t n, nr, nrp;         // nodes of the pixels' angle and of the rows' (padded to 16)
    int32_t rows, rowsp;        // pixel rows: half the detector, rounded up; padded to 16
    int32_t det_n;
    double step_r, step_i;      // exp(-i qc dz)
    const double* rot;          // [nz padded to EW_ZC] dV exp(-i qc z)
    const double* phiz;         // [nz padded to EW_ZC][kzt]
    const double* phize;        // even and odd z modes on the half axis, [(nz + 1) / 2 padded to 16]
    const double* phizo;        // x [kzet], [kzot]
    const double* phie;         // [nhMp][ket]
    const double* phio;         // [nhMp][kot]
    const double* cosN;         // [nhNp][nap]
    const double* sinN;
    const double* cm;           // [na][km][nbp]
    const double* cz;           // [na][nbp][kzp]
    const double* dcte;         // [node][k], both padded to 16: coefficient k of the even series
    const double* dcto;
    const double* wre;          // [row node][row], padded to nrp x rowsp: interpolation to the rows of
    const double* wro;          // parts even and odd in the rows' angle
    const double* tq;           // [row][column] Chebyshev argument, NaN beyond the rim
    int32_t chunk;              // nodes a whose G the forward holds at a time: na, or fewer, a multiple of 32
    int64_t offY, offS, offC, offG;   // workspace offsets in doubles (Z at 0)
};

// Host side of a plan: the sizes, and what the device tables are made from.
struct EwHost {
    bool use = false;
    EwDesc d;                                   // pointers unset
    size_t workspace = 0, adj_workspace = 0;    // bytes
    double qc = 0.0, k0 = 0.0;
    double pitchN = 0.0, pitchM = 0.0, pitchZ = 0.0;
    double limit = 0.0;                         // half-width of the screen: tan(theta) or k0 sin(theta)
    double range = 0.0;                         // largest angle of the pixels' columns
    std::vector<double> ang_a, ang_b;           // the nodes a and b
    std::vector<double> phiz, phie, phio;       // as in EwDesc
    std::vector<double> phize, phizo;           // half-axis z modes, as in EwDesc
    std::vector<double> rot, dcte, dcto, wre, wro;
};

// Fill h for the geometry (detector plans only); h->use says whether the form applies:
// its sizes lie within the limits above.  Where the forward's workspace would exceed `most`
// bytes and holding G for fewer nodes at a time keeps it below, it does.
void ew_plan(const msft_geometry& g, size_t most, EwHost* h);

// Even and odd orthonormal discrete prolate sequences of an axis of n voxels of pitch d
// for |q| <= qh, as many as hold cos(q r), sin(q r) on the voxel centres to EW_TOL of
// their norm; half[h] is the value at voxel n - 1 - h (coordinate >= 0).  limit: give
// up (false) if more than this many modes are needed.
bool ew_basis(int n, double d, double qh, int limit, int* ke, int* ko, std::vector<double>* even,
              std::vector<double>* odd);

// One request of a launch: a plan's descriptor (device memory), its buffers, and the
// pixels [p0, p1) to write.
struct EwReq {
    const EwDesc* d;
    const float* delta;
    const float* beta;
    float* intensity;
    float* amplitude;
    double* ws;
    int64_t p0, p1;
    int32_t a0;   // first node of G's part
};
struct EwOne {
    EwReq req;
    EwDesc d;   // *req.d
};
constexpr int EW_MAX_REQ = 24;
struct EwBatch {
    EwReq req[EW_MAX_REQ];
    int32_t begin[EW_MAX_REQ + 1];   // first workgroup of each request
    int32_t n;
};

// Adjoint of one request: h = g conj(A) per pixel in, gradients out.
struct EwAdj {
    const EwDesc* d;
    const float* delta;
    const float* beta;
    const float* amplitude;
    const float* grad_intensity;
    float* grad_delta;
    float* grad_beta;
    double* ws;
};

// Launchers (ewald.hip, ewald_adj.hip); dims: the host copies of the requests' descriptors.
// Device tables made on the device: cosN, sinN, cm, cz (the last two zeroed by the caller)
// from the angles and the half-axis modes dev points to.
struct EwTables {
    const double *ang_a, *ang_b;
    double *cosN, *sinN, *cm, *cz, *tq;
};
int launch_ew_tables(const EwHost& h, const EwDesc& dev, const EwTables& t, void* stream);
int launch_ew_scan(const EwBatch& b, const EwDesc* const* dims, void* stream);
int launch_ew_contract(EwBatch& b, const EwDesc* const* dims, void* stream);
int launch_ew_adjoint(const EwAdj& a, const EwDesc& dims, void* stream);

}  // namespace msft
