// Host side of the spherical-coordinate form (ewald.h): the prolate bases of the axes,
// the number of Chebyshev nodes a detector needs, and the tables made from them.
#include "ewald.h"

#include <algorithm>
#include <cmath>

#include "msft_internal.h"

namespace msft {

namespace {

constexpr double kPi = 3.14159265358979323846;

// What the truncated bases and series may leave out, relative to the norm of exp(-i q r)
// (basis) or to 1 (series).  All else is FP64 up to the FP32 outputs: 3e-11 is 2000 times below
// the rounding of a pixel at the peak, and 3e-7 of one whose intensity is 1e-8 of the peak's
// (the direct form's FP32 sums, good to 1e-7 of the peak's amplitude, leave 1e-3 there).
constexpr double EW_TOL = 3e-11;

int pad(int n, int m) { return (n + m - 1) / m * m; }

// Eigenvalues below each of four x of the symmetric tridiagonal matrix (d, off-diagonal
// squared e2), entries of order one: the sign changes of the leading minors, four chains of
// products at a time (the ratios' chains of divisions took 2.4 times as long).
void sturm_counts(const std::vector<double>& d, const std::vector<double>& e2, const double* x, int* count)
{
    constexpr double BIG = 1e150, SMALL = 1e-150;
    double p0[4], p1[4];
    int c[4];
    for (int j = 0; j < 4; ++j) {
        p0[j] = 1.0;
        p1[j] = d[0] - x[j];
        c[j] = p1[j] < 0.0;
    }
    for (size_t k = 1; k < d.size(); ++k) {
        for (int j = 0; j < 4; ++j) {
            double p = (d[k] - x[j]) * p1[j] - e2[k - 1] * p0[j];
            if (p == 0.0) p = p1[j] * 1e-30;   // no change here, one at the next
            c[j] += (p < 0.0) != (p1[j] < 0.0);
            p0[j] = p1[j];
            p1[j] = p;
        }
        if ((k & 7) == 0)   // a step grows by 3 at most and falls by 1e-7
            for (int j = 0; j < 4; ++j) {
                const double m = std::max(std::fabs(p0[j]), std::fabs(p1[j]));
                const double f = m > BIG ? SMALL : m < SMALL ? BIG : 1.0;
                p0[j] *= f;
                p1[j] *= f;
            }
    }
    for (int j = 0; j < 4; ++j) count[j] = c[j];
}

// Eigenvector of (d, e) at the eigenvalue lam: inverse iteration with a pivoted LU.
std::vector<double> tri_vector(const std::vector<double>& d, const std::vector<double>& e, double lam,
                               double scale)
{
    const int n = (int)d.size();
    if (n == 1) return {1.0};   // an axis of one or two voxels; the matrix may be zero
    std::vector<double> a(n), b(n, 0.0), c(n, 0.0), l(n, 0.0), x(n);
    std::vector<char> swapped(n, 0);
    // rows hold (diagonal, first, second superdiagonal) after elimination
    double p = d[0] - lam, q = n > 1 ? e[0] : 0.0;
    for (int k = 0; k + 1 < n; ++k) {
        const double s = e[k], dn = d[k + 1] - lam, un = k + 2 < n ? e[k + 1] : 0.0;
        if (std::fabs(p) >= std::fabs(s)) {
            if (p == 0.0) p = 1e-300;
            a[k] = p;
            b[k] = q;
            l[k] = s / p;
            p = dn - l[k] * q;
            q = un;
        } else {
            swapped[k] = 1;
            a[k] = s;
            b[k] = dn;
            c[k] = un;
            l[k] = p / s;
            p = q - l[k] * dn;
            q = -l[k] * un;
        }
    }
    a[n - 1] = std::fabs(p) > 1e-16 * scale ? p : 1e-16 * scale;
    for (double& v : a) v = 1.0 / v;
    uint32_t seed = 1;   // any start that is not orthogonal to the vector
    for (double& v : x) v = 1.0 + 1e-10 * (double)(seed = seed * 1664525u + 1013904223u);
    for (int it = 0; it < 3; ++it) {
        for (int k = 0; k + 1 < n; ++k) {
            if (swapped[k]) std::swap(x[k], x[k + 1]);
            x[k + 1] -= l[k] * x[k];
        }
        for (int k = n - 1; k >= 0; --k) {
            double v = x[k];
            if (k + 1 < n) v -= b[k] * x[k + 1];
            if (k + 2 < n) v -= c[k] * x[k + 2];
            x[k] = v * a[k];
        }
        double big = 0.0, s = 0.0;
        for (double v : x) big = std::max(big, std::fabs(v));
        big = 1.0 / big;
        for (double& v : x) {
            v *= big;
            s += v * v;
        }
        s = 1.0 / std::sqrt(s);
        for (double& v : x) v *= s;
    }
    return x;
}

// The eigenvectors of largest eigenvalue, four at a time: appends those of the eigenvalues
// ranked out->size(), ... (0 the largest); `top` lies above them and is moved down.  An
// eigenvalue is bracketed to 1e-11 of the scale, the gaps being 5.9e-7 of it or more (4095
// voxels and a narrow band; 1e-5 up to 1024 voxels): each of the three steps of the inverse
// iteration then takes nearly five digits.
struct TriTop {
    const std::vector<double>&d, &e;
    std::vector<double> ds, e2;   // over the scale, as lo and top
    double lo, top, scale;

    TriTop(const std::vector<double>& d_, const std::vector<double>& e_) : d(d_), e(e_)
    {
        const int n = (int)d.size();
        double hi = lo = d[0];
        for (int k = 0; k < n; ++k) {
            const double r = (k ? std::fabs(e[k - 1]) : 0.0) + (k + 1 < n ? std::fabs(e[k]) : 0.0);
            lo = std::min(lo, d[k] - r);
            hi = std::max(hi, d[k] + r);
        }
        scale = std::max({std::fabs(lo), std::fabs(hi), 1e-300});
        top = hi / scale + 1e-14;
        lo = lo / scale - 1e-14;
        for (double v : d) ds.push_back(v / scale);
        for (double v : e) e2.push_back(v / scale * (v / scale));
    }
    void next(std::vector<std::vector<double>>* out)
    {
        const int n = (int)d.size(), first = (int)out->size(), m = std::min(4, n - first);
        double a[4], b[4], x[4];
        int c[4];
        for (int j = 0; j < 4; ++j) {
            a[j] = lo;
            b[j] = top;
        }
        for (int it = 0; it < 200; ++it) {
            bool open = false;
            for (int j = 0; j < m; ++j) open |= b[j] - a[j] > 1e-11;
            if (!open) break;
            // the middles; of intervals that are still one, points apart
            const bool one = a[0] == a[3] && b[0] == b[3];
            for (int j = 0; j < 4; ++j) x[j] = a[j] + (one ? 0.2 * (j + 1) : 0.5) * (b[j] - a[j]);
            sturm_counts(ds, e2, x, c);
            // every count bounds every one of the eigenvalues n - 1 - first - j
            for (int j = 0; j < m; ++j)
                for (int i = 0; i < 4; ++i) {
                    if (c[i] >= n - first - j) b[j] = std::min(b[j], x[i]);
                    else a[j] = std::max(a[j], x[i]);
                }
        }
        for (int j = 0; j < m; ++j) out->push_back(tri_vector(d, e, 0.5 * (a[j] + b[j]) * scale, scale));
        top = b[m - 1];   // above the next one: b only falls on counts that hold it
    }
};

// Terms after which the Chebyshev series of exp(i (x sin(w t) + s r cos(w t))) over |t| <= 1,
// w at most pi / 2, is below EW_TOL, the largest of three shares s of r.  Any count from
// `enough` on stands for more; 0: more than a plan is planned for.
int series_terms(double x, double r, double w, int enough)
{
    const double reach = (x + r) * w;
    if (reach + 14.0 * std::cbrt(reach) + 40.0 > 6.0 * EW_MAX_NODES + 1.0) return 0;
    // with t = cos(theta) the terms are a Fourier series, which goes on to the phase's largest
    // rate in theta and falls off within some cube roots of it
    double rate = 0.0;
    for (int k = 0; k < 64; ++k) {
        const double th = (k + 0.5) * kPi / 128.0, a = w * std::cos(th);
        rate = std::max(rate, w * (x * std::cos(a) + r * std::sin(a)) * std::sin(th));
    }
    if (rate >= enough) return enough;
    int worst = 1;
    std::vector<double> cs, er, ei, odr, odi;
    for (int M = pad((int)(rate + 10.0 * std::cbrt(rate * (1.0 + w * w))) + 16, 8);; M = pad(M + M / 2, 8)) {
        const int half = M / 2;   // nodes of t > 0; those at -t add the same or nothing
        cs.resize(4 * M);
        for (int k = 0; k < 4 * M; ++k) cs[k] = std::cos(kPi * k / (2.0 * M));
        for (auto* v : {&er, &ei, &odr, &odi}) v->resize(half);
        bool ended = true;
        worst = 1;
        for (double s : {0.0, 0.5, 1.0}) {
            for (int j = 0; j < half; ++j) {   // the even and the odd part in t
                const double a = w * cs[2 * j + 1], p = x * std::sin(a), q = s * r * std::cos(a);
                const double cp = std::cos(p), sp = std::sin(p), cq = std::cos(q), sq = std::sin(q);
                er[j] = cq * cp;
                ei[j] = sq * cp;
                odr[j] = -sq * sp;
                odi[j] = cq * sp;
            }
            // coefficients from the highest down, until their sum is too much to leave out
            double tail = 0.0;
            int need = M;
            for (; need > worst; --need) {
                const int k = need - 1;
                const double *fr = (k & 1 ? odr : er).data(), *fi = (k & 1 ? odi : ei).data();
                double re = 0.0, im = 0.0;
                for (int j = 0, at = k; j < half; ++j) {
                    re += fr[j] * cs[at];
                    im += fi[j] * cs[at];
                    at += 2 * k;
                    if (at >= 4 * M) at -= 4 * M;
                }
                tail += 4.0 / M * std::sqrt(re * re + im * im);
                if (tail >= EW_TOL) break;
                if (need == M - 7) ended &= tail < 1e-2 * EW_TOL;
            }
            ended &= need <= M - 8;   // else more nodes: the series goes on past M
            worst = std::max(worst, need);
        }
        if (ended) return worst;
    }
}

}  // namespace

bool ew_basis(int n, double d, double qh, int limit, int* ke, int* ko, std::vector<double>* even,
              std::vector<double>* odd)
{
    const int nh = (n + 1) / 2, m = n / 2;
    const double W = std::min(qh * d / (2.0 * kPi), 0.5);
    if (2.0 * n * W > (double)limit) return false;
    // the tridiagonal matrix that commutes with the band limit of [-W, W] (Slepian 1978)
    const double cw = std::cos(2.0 * kPi * W);
    auto diag = [&](int k) { return 0.25 * (n - 1.0 - 2.0 * k) * (n - 1.0 - 2.0 * k) * cw; };
    auto off = [&](int k) { return 0.5 * k * (double)(n - k); };   // couples k - 1 and k
    const double share[] = {0.0, 0.25, 0.5, 0.7, 0.85, 0.93, 0.97, 0.99, 1.0};
    for (int par = 0; par < 2; ++par) {
        std::vector<double>& out = par ? *odd : *even;
        int& kept = par ? *ko : *ke;
        kept = 0;
        out.clear();
        // even or odd half of the matrix (an odd n's centre enters the even half with sqrt 2)
        const int size = (n % 2 && par == 0) ? m + 1 : m;
        if (size == 0) continue;
        std::vector<double> td(size), te(std::max(size - 1, 0));
        for (int k = 0; k < size; ++k) td[k] = diag(k);
        for (int k = 0; k + 1 < size; ++k) te[k] = off(k + 1);
        if (n % 2 == 0) td[size - 1] += par ? -off(m) : off(m);
        else if (par == 0 && size > 1) te[size - 2] *= std::sqrt(2.0);
        // residual of cos or sin(q r) after the first K modes, over sample momenta
        std::vector<std::vector<double>> v, res;
        for (double s : share) {
            std::vector<double> r(nh);
            for (int h = 0; h < nh; ++h) {
                const double ph = s * qh * (n - 1.0 - 2.0 * h) * d / 2.0;
                r[h] = par ? std::sin(ph) : std::cos(ph);
            }
            res.push_back(r);
        }
        TriTop tri(td, te);
        const int least = (int)(n * W) - 1;   // half the modes concentrated in the band
        int K = 0;
        for (; K < size; ++K) {
            double worst = 0.0;
            if (K >= least)
                for (auto& r : res) {
                    double s = 0.0;
                    for (int h = 0; h < nh; ++h) s += (n % 2 && h == m ? 1.0 : 2.0) * r[h] * r[h];
                    worst = std::max(worst, s);
                }
            if (K >= least && std::sqrt(worst / n) < EW_TOL) break;
            if (K == (int)v.size()) {
                tri.next(&v);
                for (size_t j = K; j < v.size(); ++j) {
                    for (int k = 0; k < size; ++k)
                        if (!(n % 2 && k == m)) v[j][k] *= std::sqrt(0.5);
                    v[j].resize(nh, 0.0);
                }
            }
            for (auto& r : res) {
                double c = 0.0;
                for (int h = 0; h < nh; ++h) c += (n % 2 && h == m ? 1.0 : 2.0) * r[h] * v[K][h];
                for (int h = 0; h < nh; ++h) r[h] -= c * v[K][h];
            }
        }
        kept = K;
        out.assign((size_t)nh * K, 0.0);
        for (int k = 0; k < K; ++k)
            for (int h = 0; h < nh; ++h) out[(size_t)h * K + k] = v[k][h];
    }
    return *ke + *ko <= limit;
}

void ew_plan(const msft_geometry& g, size_t most_bytes, EwHost* hp)
{
    EwHost& H = *hp;
    EwDesc& d = H.d;
    d = EwDesc{};
    H.use = false;
    const int N = g.det_n, half = (N + 1) / 2;
    const double k0 = (2.0 * kPi) / g.wavelength, theta = (g.theta_max_deg * kPi) / 180.0;
    const double hx = 0.5 * (g.nx - 1) * g.dx, hy = 0.5 * (g.ny - 1) * g.dy, hz = 0.5 * (g.nz - 1) * g.dz;
    const bool uni = g.flags & MSFT_DETECTOR_UNIFORM_Q;
    d.uniform = uni;
    d.det_n = N;
    d.rows = half;
    d.rowsp = pad(half, 16);
    H.k0 = k0;
    // the rows' angle, and the largest of the pixels' other one, at non-negative coordinates
    // (index N - 1 - h); its tangent is u cos b (flat) or q_x / sqrt(k0^2 - q_x^2 - q_y^2)
    std::vector<double> pos(half), row(half);
    H.limit = uni ? k0 * std::sin(theta) : std::tan(theta);
    for (int h = 0; h < half; ++h) {
        pos[h] = ((double)(N - 1 - 2 * h) * H.limit) / (double)N;
        row[h] = uni ? std::asin(std::min(1.0, pos[h] / k0)) : std::atan(pos[h]);
    }
    double range = 0.0;
    if (uni) {
        const double kk = k0 * k0;
        double ratio = -1.0, x = 0.0, z = 1.0;
        for (int j = 0; j < half; ++j)
            for (int i = 0; i < half; ++i) {
                const double s = pos[i] * pos[i] + pos[j] * pos[j];
                if (!(s < kk)) continue;
                if (pos[i] * pos[i] > ratio * (kk - s)) {
                    ratio = pos[i] * pos[i] / (kk - s);
                    x = pos[i];
                    z = kk - s;
                }
                break;   // the widest pixel of a row within the rim is its first
            }
        range = std::atan2(x, std::sqrt(z));
    } else {
        for (double b : row) range = std::max(range, std::atan(pos[0] * std::cos(b)));
    }
    H.range = range;
    const double rrange = row[0];
    // largest M sin b + z cos b of the box over |b| <= w: what exp(-i q r) holds beside N sin a
    const double hN = uni ? hy : hx, hM = uni ? hx : hy, wb = uni ? range : rrange;
    const double top = std::atan2(hM, hz), r = top <= wb ? std::hypot(hM, hz) : hM * std::sin(wb) + hz * std::cos(wb);
    const double wa = uni ? rrange : range;
    // past the limit of the pixels' angle, or as many as the rows, the count does not matter
    const int enough[] = {2 * half, 2 * EW_MAX_NODES + 1};
    const int ta = wa > 0.0 ? series_terms(k0 * hN, k0 * r, wa, enough[!uni]) : 1;
    if (ta == 0 || (!uni && ta > 2 * EW_MAX_NODES)) return;
    const int tb = wb > 0.0 ? series_terms(k0 * hM, k0 * hz, wb, enough[uni]) : 1;
    const int n = ((uni ? tb : ta) + 1) / 2;
    int nr = ((uni ? ta : tb) + 1) / 2;
    if (tb == 0 || n > EW_MAX_NODES) return;
    const bool exact = nr >= half;   // no more rows than nodes: the rows themselves
    if (exact) nr = half;
    if (nr > EW_MAX_NODES) return;
    d.n = n;
    d.nr = nr;
    d.nrp = pad(nr, 16);
    std::vector<double> col(n);
    std::vector<double> rn(row);
    for (int k = 0; k < n; ++k) col[k] = range * std::cos((k + 0.5) * kPi / (2.0 * n));
    if (!exact) {
        rn.resize(nr);
        for (int k = 0; k < nr; ++k) rn[k] = rrange * std::cos((k + 0.5) * kPi / (2.0 * nr));
    }
    H.ang_a = uni ? rn : col;
    H.ang_b = uni ? col : rn;
    // values at the rows from values at the row nodes: Lagrange's polynomials of the 2 nr
    // Chebyshev points in barycentric form, those of +- a node folded for even and odd parts
    H.wre.assign((size_t)d.nrp * d.rowsp, 0.0);
    H.wro.assign((size_t)d.nrp * d.rowsp, 0.0);
    constexpr int JB = 8;   // rows at a time: their weights are neighbours
    std::vector<double> nodes(nr), weights(nr), pole(JB * nr);
    for (int k = 0; k < nr; ++k) {
        const double w = (k + 0.5) * kPi / (2.0 * nr);
        nodes[k] = std::cos(w);
        weights[k] = (k & 1 ? -2.0 : 2.0) * std::sin(w);
    }
    for (int j0 = 0; j0 < half; j0 += JB) {
        const int rows = std::min(JB, half - j0);
        if (exact) {
            for (int j = j0; j < j0 + rows; ++j) H.wre[(size_t)j * d.rowsp + j] = H.wro[(size_t)j * d.rowsp + j] = 1.0;
            continue;
        }
        // s / (t - x) at x and, of the other sign, at -x (point 2 nr - 1 - k): sum and difference
        double t[JB], scale[JB];
        int hit[JB];
        for (int u = 0; u < rows; ++u) {
            t[u] = row[j0 + u] / rrange;
            hit[u] = -1;
            double sum = 0.0;
            for (int k = 0; k < nr; ++k) {
                const double x = nodes[k];
                if (t[u] == x) hit[u] = k;
                pole[JB * k + u] = weights[k] / ((t[u] - x) * (t[u] + x));
                sum += pole[JB * k + u] * x;
            }
            scale[u] = 1.0 / sum;
        }
        for (int k = 0; k < nr; ++k)
            for (int u = 0; u < rows; ++u) {
                const double p = pole[JB * k + u] * scale[u];
                H.wre[(size_t)k * d.rowsp + j0 + u] = hit[u] >= 0 ? (double)(k == hit[u]) : p * nodes[k];
                H.wro[(size_t)k * d.rowsp + j0 + u] = hit[u] >= 0 ? (double)(k == hit[u]) : p * t[u];
            }
    }
    d.na = (int)H.ang_a.size();
    d.nb = (int)H.ang_b.size();
    d.nap = pad(d.na, 16);
    d.nbp = pad(d.nb, 16);
    // momentum ranges over all (a, b)
    double qm = 0.0, zlo = 0.0, zhi = -2.0 * k0;
    std::vector<double> sb2, sbn;   // sin^2(b/2), |sin b|
    double sa2 = 0.0, ca = 1.0;
    for (double b : H.ang_b) {
        sb2.push_back(std::sin(0.5 * b) * std::sin(0.5 * b));
        sbn.push_back(std::fabs(std::sin(b)));
    }
    for (double a : H.ang_a)
        for (size_t b = 0; b < sb2.size(); ++b) {
            if (b == 0) {
                sa2 = std::sin(0.5 * a) * std::sin(0.5 * a);
                ca = std::cos(a);
            }
            const double qz = -2.0 * k0 * (sa2 + ca * sb2[b]);
            qm = std::max(qm, k0 * std::fabs(ca) * sbn[b]);
            zlo = std::min(zlo, qz);
            zhi = std::max(zhi, qz);
        }
    H.qc = 0.5 * (zlo + zhi);
    H.pitchN = uni ? g.dy : g.dx;
    H.pitchM = uni ? g.dx : g.dy;
    H.pitchZ = g.dz;
    d.nx = g.nx;
    d.ny = g.ny;
    d.nz = g.nz;
    d.strength = g.strength;
    d.k0dz64 = k0 * g.dz;
    d.dV64 = g.dx * g.dy * g.dz;
    d.step_r = std::cos(H.qc * g.dz);
    d.step_i = -std::sin(H.qc * g.dz);
    d.nN = uni ? g.ny : g.nx;
    d.nM = uni ? g.nx : g.ny;
    d.zsN = uni ? 1 : g.ny;
    d.zsM = uni ? g.ny : 1;
    d.nhN = (d.nN + 1) / 2;
    d.nhM = (d.nM + 1) / 2;
    d.nhNp = pad(d.nhN, 16);
    d.nhMp = pad(d.nhM, 16);
    std::vector<double> ze, zo, me, mo;
    int kze, kzo, ke, ko;
    if (!ew_basis(g.nz, g.dz, 0.5 * (zhi - zlo), EW_MAX_KZ, &kze, &kzo, &ze, &zo)) return;
    if (!ew_basis(d.nM, H.pitchM, qm, EW_MAX_KM, &ke, &ko, &me, &mo)) return;
    d.kze = kze;
    d.kz = kze + kzo;
    d.kzp = pad(d.kz, 4);
    d.kzt = pad(d.kz, 16);
    d.ld = 2 * d.kzp;
    d.kep = pad(ke, 4);
    d.kop = pad(ko, 4);
    d.km = d.kep + d.kop;
    d.ket = pad(ke, 16);
    d.kot = pad(std::max(ko, 1), 16);
    // tables
    const int nzp = pad(g.nz, EW_ZC), nhz = (g.nz + 1) / 2;
    H.rot.assign(2 * (size_t)nzp, 0.0);
    H.phiz.assign((size_t)nzp * d.kzt, 0.0);
    for (int z = 0; z < g.nz; ++z) {
        const double ph = H.qc * (((double)(2 * z + 1 - g.nz) * g.dz) / 2.0);
        H.rot[2 * z] = d.dV64 * std::cos(ph);
        H.rot[2 * z + 1] = -d.dV64 * std::sin(ph);
        const int h = std::min(z, g.nz - 1 - z);
        const double sign = 2 * z + 1 >= g.nz ? 1.0 : -1.0;
        for (int l = 0; l < kze; ++l) H.phiz[(size_t)z * d.kzt + l] = ze[(size_t)h * kze + l];
        for (int l = 0; l < kzo; ++l) H.phiz[(size_t)z * d.kzt + kze + l] = sign * zo[(size_t)h * kzo + l];
    }
    d.kzet = pad(kze, 16);
    d.kzot = pad(std::max(kzo, 1), 16);
    H.phize.assign((size_t)pad(nhz, 16) * d.kzet, 0.0);
    H.phizo.assign((size_t)pad(nhz, 16) * d.kzot, 0.0);
    for (int h = 0; h < nhz; ++h) {
        for (int l = 0; l < kze; ++l) H.phize[(size_t)h * d.kzet + l] = ze[(size_t)h * kze + l];
        for (int l = 0; l < kzo; ++l) H.phizo[(size_t)h * d.kzot + l] = zo[(size_t)h * kzo + l];
    }
    H.phie.assign((size_t)d.nhMp * d.ket, 0.0);
    H.phio.assign((size_t)d.nhMp * d.kot, 0.0);
    for (int h = 0; h < d.nhM; ++h) {
        for (int m = 0; m < ke; ++m) H.phie[(size_t)h * d.ket + m] = me[(size_t)h * ke + m];
        for (int m = 0; m < ko; ++m) H.phio[(size_t)h * d.kot + m] = mo[(size_t)h * ko + m];
    }
    const int np = pad(n, 16);
    H.dcte.assign((size_t)np * np, 0.0);
    H.dcto.assign((size_t)np * np, 0.0);
    std::vector<double> turn(8 * n);   // cos(j pi / (4 n))
    for (int j = 0; j < 8 * n; ++j) turn[j] = std::cos(j * kPi / (4.0 * n));
    for (int a = 0; a < n; ++a)
        for (int k = 0; k < n; ++k) {   // at the angles (a + 1/2) pi / (2 n) times 2 k and 2 k + 1
            H.dcte[(size_t)a * np + k] = (k ? 2.0 : 1.0) / n * turn[(2 * a + 1) * 2 * k % (8 * n)];
            H.dcto[(size_t)a * np + k] = 2.0 / n * turn[(2 * a + 1) * (2 * k + 1) % (8 * n)];
        }
    // workspace: Z is kept for a second contraction, so nothing shares its place
    const int64_t z = (int64_t)g.nx * g.ny * d.ld, y = (int64_t)d.nN * d.km * d.ld;
    const int64_t node = 2 * (int64_t)d.km * d.ld;   // G of one node
    auto up = [](int64_t v) { return (v + 31) / 32 * 32; };
    d.offY = up(z);
    d.offS = d.offY + up(y);
    d.offC = d.offS + up((int64_t)d.nr * n * 8);
    d.offG = d.offC + up((int64_t)d.rows * n * 8);
    d.chunk = d.na;
    H.adj_workspace = H.workspace = (size_t)(d.offG + up(node * d.na)) * 8;
    const int64_t left = ((int64_t)(most_bytes / 8) - d.offG) / node / 32 * 32;
    if (H.workspace > most_bytes && left > 0) {
        const int parts = (int)((d.na + left - 1) / left);
        d.chunk = pad((d.na + parts - 1) / parts, 32);
        H.workspace = (size_t)(d.offG + up(node * d.chunk)) * 8;
    }
    H.use = true;
}

}  // namespace msft
