// Which form a detector plan's forward and adjoint take: estimates of both forms' times.
//
// The constants (us) are least-squares fits to 940 random plans timed on an MI355X: voxel
// counts 1 to 4096 an axis, sides 1 to 1024, both detectors, FP32 and the split; nine
// estimates in ten lie within a third of the time measured.  What they have to catch are
// few pixels (64 on 256^3 voxels at 16 nm: gradient 749 us in the spherical form, whose
// angles go by the grid alone, 390 direct; over half of the gradients of sides below 32 were
// slower), few columns of more than EW_WHOLE_NZ slices (14 x 2 x 1734 on 109^2,
// split: 1102 against 242), and uniform plans of many angles (333 x 87 x 64 on 78^2:
// gradient 278 against 53).
//
// The form's results are some 4 (FP32) to 40 times (split) nearer to the 64-bit values, so it
// is left only where the direct form is faster by a margin: 1.25 (few of the plans sent away by
// it were faster in the form, the worst by 1.4), but 2 on the uniform detector up to
// EW_WHOLE_NZ slices, where the direct form is itself a separable one and within a factor of two
// of the other over much of the range.
#include <algorithm>

#include "msft_internal.h"

namespace msft {

namespace {

constexpr double MARGIN = 1.25, MARGIN_UNIFORM = 2.0;

template <int N>
double dot(const double (&c)[N], const double (&x)[N])
{
    double s = 0.0;
    for (int k = 0; k < N; ++k) s += c[k] * x[k];
    return s;
}

struct Times {
    double forward, adjoint;
};

// One workgroup walks all W tiles, two of them to a CU in FP32; the adjoint's groups of pixels
// walk theirs in chunks of ADJ_CHUNK, one workgroup to a CU, and write partial sums.
Times direct_flat(const msft_plan_s* p)
{
    const Dims& d = p->dims;
    const AdjDims a = make_adj_dims(d);
    const bool fp32 = p->geo.g.precision == MSFT_FP32;
    const double tiles = (double)d.ntiles(), voxels = (double)d.nx * d.ny * d.nz;
    const double waves = (double)ceil_div(d.nblocks, fp32 ? 2 * CHIP_CUS : CHIP_CUS);
    const double chunks = (double)a.group_pix / ADJ_CHUNK, groups = (double)d.nxc * d.nzb * a.nyb * a.nsplit;
    const double x[] = {1.0, tiles * waves, tiles, std::min(tiles, 100.0)};
    const double y[] = {1.0, chunks, chunks * groups / CHIP_CUS, a.rpart_bytes * 1e-6, (double)ceil_div(d.nz, 64),
                        voxels * 1e-6};
    const double f32[] = {24.7, 1.395, 0.0, 0.329}, split[] = {22.5, 0.428, 0.471, 0.269};
    const double adj[] = {10.1, 11.3, 19.8, 0.386, 1.61, 6.46};
    return {fp32 ? dot(f32, x) : dot(split, x), dot(adj, y)};
}

// Forward: stage 2's workgroup walks the (y chunk, z block) tiles of its columns, stage 1's the
// x chunks; adjoint: the rows' pass, the columns' pass, the walk.
Times direct_uniform(const msft_plan_s* p)
{
    const Dims& d = p->dims;
    const bool fp32 = p->geo.g.precision == MSFT_FP32;
    const int64_t n = p->sep.n, chunk = fp32 ? 32 : 64;
    const double yz = (double)ceil_div(d.ny, chunk) * d.nzb, xc = (double)ceil_div(d.nx, chunk);
    const double blocks = (double)ceil_div(n, BLOCK_PIX), ic = (double)ceil_div(n, 32), cus = (double)CHIP_CUS;
    const double voxels = (double)d.nx * d.ny * d.nz;
    const double x[] = {1.0, yz, yz * n * blocks / cus, xc, xc * d.ny * d.nzb * blocks / cus, n * yz * 1e-3};
    const double y[] = {1.0, ic, ic * ceil_div(d.ny, 16) * n * d.nzb * 1e-4,
                        ic * ceil_div(d.nx, 32) * d.ny * d.nzb * 1e-3, voxels * 1e-6, (double)ceil_div(d.nz, 64)};
    const double f32[] = {16.3, 1.48, 2.10, 5.01, 2.54, 0.0}, split[] = {16.5, 1.35, 2.20, 5.87, 1.41, 5.86};
    const double a32[] = {15.2, 2.35, 19.4, 2.25, 16.5, 2.42}, asplit[] = {13.5, 7.83, 21.6, 3.36, 7.67, 10.2};
    return {fp32 ? dot(f32, x) : dot(split, x), fp32 ? dot(a32, y) : dot(asplit, y)};
}

// The launches, the voxels, rounds of long columns (768 workgroups at once), products of the
// modal and nodes stages, those of the scan, tables and G, nodes, pixels.
Times spherical(const EwDesc& d)
{
    const double columns = (double)d.nx * d.ny, voxels = columns * d.nz, modes = (double)d.km * d.ld;
    const double rounds = ew_rounds(d.nz) ? 0.0 : (double)ceil_div(d.nz, EW_ZC) * std::max(1.0, columns / EW_COLS / 768.0);
    const double x[] = {1.0, voxels * 1e-6, rounds, modes * (columns + 2.0 * d.na * d.nhN) * 1e-9, voxels * d.kz * 1e-9,
                        d.na * (8.0 * d.nbp * (d.km + d.kzp) + 16.0 * modes) * 1e-6, (double)d.n,
                        (double)d.det_n * d.det_n * 1e-6};
    const double fwd[] = {21.2, 3.42, 18.0, 35.4, 118.0, 0.843, 0.106, 4.79};
    const double adj[] = {17.3, 4.20, 4.49, 119.0, 217.0, 1.03, 0.280, 57.1};
    return {dot(fwd, x), dot(adj, x)};
}

}  // namespace

void choose_forms(const msft_plan_s* p, bool* forward, bool* adjoint)
{
    const Times e = spherical(p->ew.d), d = p->separable ? direct_uniform(p) : direct_flat(p);
    const double margin = p->separable && p->dims.nz <= EW_WHOLE_NZ ? MARGIN_UNIFORM : MARGIN;
    *forward = e.forward <= margin * d.forward;
    *adjoint = e.adjoint <= margin * d.adjoint;
}

}  // namespace msft
