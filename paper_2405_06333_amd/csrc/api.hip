// C ABI of librbe2d (declared in include/rbe2d.h): parameter validation,
// derived constants, workspace management, the host k-sampler, layouts of
// one or many systems, and the launch sequences of one RBE2D evaluation
// (Algorithm 2 of the paper) and of velocity-Verlet steps around it.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "rbe2d_internal.h"

// cells per r_c along y of the FP32 pair kernel's cell grid
#ifndef RBE2D_REACH_Y
#define RBE2D_REACH_Y 6
#endif

using namespace rbe2d;

namespace {

thread_local std::string g_create_error;

rbe2d_status fail(rbe2d_ctx *h, rbe2d_status st, const char *fmt, ...) __attribute__((format(printf, 3, 4)));
rbe2d_status fail(rbe2d_ctx *h, rbe2d_status st, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h) h->err = buf; else g_create_error = buf;
    return st;
}

rbe2d_status hipfail(rbe2d_ctx *h, hipError_t e, const char *what) {
    return fail(h, RBE2D_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define RBE2D_TRY(h, call, what)                           \
    do {                                                   \
        hipError_t e_ = (call);                            \
        if (e_ != hipSuccess) return hipfail(h, e_, what); \
    } while (0)

bool finite_pos(double x) { return std::isfinite(x) && x > 0.0; }

double ipow(double b, int e) {
    double r = 1.0;
    for (int i = 0; i < e; i++) r *= b;
    return r;
}

// exponents (a of gamma_top, b of gamma_bot) of the order-l image above (+1) or below (-1)
void exponents(int l, int side, int *a, int *b) {
    const int up = (l + 1) / 2, dn = l / 2;
    if (side > 0) { *a = up; *b = dn; } else { *a = dn; *b = up; }
}

double dmono(int e_self, double g_self, int e_other, double g_other) {
    return e_self ? e_self * ipow(g_self, e_self - 1) * ipow(g_other, e_other) : 0.0;
}

// one-axis theta factor of S: sum_n exp(-pi^2 n^2 / (alpha L)^2)
double theta_axis(double alpha, double L) {
    double s = 1.0;
    for (long n = 1;; n++) {
        const double t = std::exp(-(kPi * kPi) * (double)(n * n) / (alpha * alpha * L * L));
        if (t < 1e-300) break;
        s += 2.0 * t;
    }
    return s;
}

// inverse-CDF table of one axis of the k-distribution, |n| <= nmax
void axis_table(double alpha, double L, int *nmax, std::vector<double> &cdf) {
    const double sig10 = 10.0 * alpha * L / (std::sqrt(2.0) * kPi);
    *nmax = (int)std::ceil(sig10) + 1;
    const int n = 2 * *nmax + 1;
    cdf.assign(n, 0.0);
    double acc = 0.0;
    for (int m = 0; m < n; m++) {
        const long v = m - *nmax;
        acc += std::exp(-(kPi * kPi) * (double)(v * v) / (alpha * alpha * L * L));
        cdf[m] = acc;
    }
    for (int m = 0; m < n; m++) cdf[m] /= acc;
}

rbe2d_status validate(const rbe2d_params *p, rbe2d_ctx *h) {
    if (!p) return fail(h, RBE2D_E_INVAL, "params is NULL");
    if (!finite_pos(p->Lx) || !finite_pos(p->Ly) || !finite_pos(p->H))
        return fail(h, RBE2D_E_INVAL, "Lx, Ly, H must be finite and > 0");
    if (!(std::fabs(p->gamma_top) <= 1.0) || !(std::fabs(p->gamma_bot) <= 1.0))
        return fail(h, RBE2D_E_INVAL, "|gamma_top|, |gamma_bot| must be <= 1");
    if (!finite_pos(p->alpha)) return fail(h, RBE2D_E_INVAL, "alpha must be finite and > 0");
    if (!finite_pos(p->r_c) || p->r_c > 0.5 * std::min(p->Lx, p->Ly))
        return fail(h, RBE2D_E_INVAL, "r_c must satisfy 0 < r_c <= min(Lx, Ly)/2");
    if (p->P < 1 || p->P > 65536) return fail(h, RBE2D_E_INVAL, "P must be in [1, 65536]");
    if (p->M < 0 || p->M > 64) return fail(h, RBE2D_E_INVAL, "M must be in [0, 64]");
    if (p->precision != RBE2D_PREC_FP64 && p->precision != RBE2D_PREC_FP32_PHASE)
        return fail(h, RBE2D_E_INVAL, "unknown precision %d", p->precision);
    if (p->reserved != 0) return fail(h, RBE2D_E_INVAL, "reserved must be 0");
    if (p->n_max < 0 || p->n_max > (int64_t)1 << 30)
        return fail(h, RBE2D_E_INVAL, "n_max must be in [0, 2^30]");
    if (!std::isfinite(p->Lz_ext) || !std::isfinite(p->eps_lz) || !std::isfinite(p->coulomb_prefactor))
        return fail(h, RBE2D_E_INVAL, "non-finite parameter");
    if (p->eps_lz >= 1.0) return fail(h, RBE2D_E_INVAL, "eps_lz must be < 1");
    return RBE2D_OK;
}

double auto_lz(const rbe2d_params *p) {
    const double eps = p->eps_lz > 0.0 ? p->eps_lz : 1e-6;
    const double lg = std::log(1.0 / eps);
    return (p->M + 1) * p->H + std::max(std::max(p->Lx, p->Ly) / (2.0 * kPi) * lg, std::sqrt(lg) / p->alpha);
}

// Cell grid of the FP32 pair kernel: cells >= r_c / reach in x (searched
// +-reach columns), layers >= r_c / 2 in z and cells >= r_c / reach_y along y,
// where the kernel scans contiguous runs of cells (finer cells trim the runs'
// ends); coarsened if there would be too many cells.  Where a cutoff sphere
// holds few particles (n_max / volume * r_c^3 < 20) the runs are short and
// their set-up dominates: x-cells of r_c (three columns), and at most two
// layers in a slab thinner than 2 r_c (measured on the 64-replica batch: 4 %
// faster steps than r_c / 2 in both)
void scan_grid(const rbe2d_params &p, SysDesc &d, int *pncx, int *pncy, int *pncz) {
    const double per_rc3 = (double)p.n_max / (p.Lx * p.Ly * p.H) * p.r_c * p.r_c * p.r_c;
    d.reach = per_rc3 < 20.0 ? 1 : 2;
    d.reach_y = RBE2D_REACH_Y;
    int ncx = std::max(1, (int)std::floor(d.reach * p.Lx / p.r_c));
    int ncy = std::max(1, (int)std::floor(d.reach_y * p.Ly / p.r_c));
    int ncz = std::max(1, (int)std::floor(2.0 * p.H / p.r_c));
    if (per_rc3 < 20.0 && p.H < 2.0 * p.r_c) ncz = std::min(ncz, 2);
    const int64_t cell_cap = std::max<int64_t>(2 * p.n_max, 4096);
    while ((int64_t)ncx * ncy * ncz > cell_cap && (ncx > 5 || ncy > 5 || ncz > 1)) {
        if (ncz > 1) ncz = (ncz + 1) / 2;
        else { ncx = std::max(5, ncx / 2); ncy = std::max(5, ncy / 2); }
    }
    *pncx = ncx; *pncy = ncy; *pncz = ncz;
}

// Cell grid of the tile kernel (FP64).  A tile of 64 targets fills a stretch of a
// column (x-cell and z-layer); its candidates are the columns within r_c, cut
// along y.  Wide columns make short tiles but include more of the slab around
// them, narrow ones make long tiles and many runs: the expected candidates and
// runs of a tile are added up for a few widths, in instructions (about 150 per
// chunk of 64 candidates, 12 per run), and the cheapest is taken.  (1e6-ion
// slab: columns of r_c in x and z, 1390 candidates and 12 runs per tile against
// 2010 and 43 for r_c / 2.)  Along y a cell is r_c / 6 or holds about 6
// particles, whichever is finer: cells bound the ends of the runs, and
// particles are ranked within them.
void tile_grid(const rbe2d_params &p, bool images, int *ncx, int *ncy, int *ncz) {
    const double rc = p.r_c, rho = std::max<double>(1.0, (double)p.n_max) / (p.Lx * p.Ly * p.H);
    auto cells_y = [&](int nx, int nz) {
        const double hy = std::min(rc / 6.0, 6.0 / (rho * (p.Lx / nx) * (p.H / nz)));
        return std::max(1.0, std::min(1e6, std::floor(p.Ly / hy)));
    };
    double best = 1e300;
    *ncx = *ncy = *ncz = 1;
    for (double f : {0.5, 0.75, 1.0, 1.5, 2.0, 3.0}) {
        const int nx = (int)std::max(1.0, std::min(1e6, std::floor(p.Lx / (f * rc))));
        const int nz_max = (int)std::max(1.0, std::min(32.0, std::ceil(2.0 * p.H / rc)));
        for (int nz = 1; nz <= nz_max; nz++) {
            const double hx = p.Lx / nx, hz = p.H / nz, hy = p.Ly / cells_y(nx, nz);
            const double stretch = 64.0 / (rho * hx * hz), len = std::min(stretch, p.Ly);
            const double columns = std::max(1.0, stretch / p.Ly);   // of the tile itself
            double cand = 0.0, runs = 0.0;
            for (int l = 0; l < nz; l++)
                for (int m = images ? -nz : 0; m < (images ? 2 * nz : nz); m++) {
                    const double dz = std::max(0, std::abs(m - l) - 1) * hz;
                    if (dz >= rc) continue;
                    for (int i = 0; i == 0 || (i - 1) * hx < rc; i++) {
                        const double dx = std::max(0, i - 1) * hx, y2 = rc * rc - dx * dx - dz * dz;
                        if (y2 <= 0.0) continue;
                        const double n = i == 0 ? columns : 2.0;
                        cand += n * rho * hx * hz * (len + 2.0 * std::sqrt(y2) + hy);
                        runs += n;
                    }
                }
            const double cost = (cand / 64.0 * 150.0 + runs * 12.0) / nz;
            if (cost < best) { best = cost; *ncx = nx; *ncz = nz; }
        }
    }
    *ncy = (int)cells_y(*ncx, *ncz);
    // no more cells than the workspace plan allows for this many particles
    const int64_t cap = std::max<int64_t>(2 * p.n_max, 4096);
    while ((int64_t)*ncx * *ncy * *ncz > cap) {
        int *big = *ncx > *ncy ? ncx : ncy;
        if (*ncz > *big) big = ncz;
        *big = (*big + 1) / 2;
    }
}

void surface_setup(SysHost &sh);

// Derived constants, image tables, real-space families, sampler tables and
// cell grid of one system.
rbe2d_status setup_system(const rbe2d_params *pin, SysHost &sh) {
    rbe2d_status st = validate(pin, nullptr);
    if (st) return st;
    sh.p = *pin;
    rbe2d_params &p = sh.p;
    SysDesc &d = sh.d;
    std::memset(&d, 0, sizeof d);
    if (p.eps_lz <= 0.0) p.eps_lz = 1e-6;
    if (p.coulomb_prefactor == 0.0) p.coulomb_prefactor = 1.0;
    const double Lz = p.Lz_ext > 0.0 ? p.Lz_ext : auto_lz(&p);
    if (Lz < (p.M + 1) * p.H)
        return fail(nullptr, RBE2D_E_INVAL,
                    "Lz_ext = %g < (M+1) H = %g: the z-replicas of the charges would overlap their images",
                    p.Lz_ext, (p.M + 1) * p.H);
    p.Lz_ext = Lz;
    d.Lx = p.Lx; d.Ly = p.Ly; d.H = p.H; d.Lz = Lz;
    d.V = p.Lx * p.Ly * Lz;
    d.S = theta_axis(p.alpha, p.Lx) * theta_axis(p.alpha, p.Ly) * theta_axis(p.alpha, Lz) - 1.0;
    d.alpha = p.alpha; d.rc = p.r_c; d.rc2 = p.r_c * p.r_c; d.pref = p.coulomb_prefactor;
    d.rc_lay = p.r_c + 1e-9 * p.r_c;   // the margin covers the division that assigned the layers
    d.H_rc = p.H + p.r_c;
    d.g_top = p.gamma_top; d.g_bot = p.gamma_bot; d.M = p.M;
    d.cfac = 2.0 * kPi * d.S * d.pref / (d.V * p.P);

    // image weights, their derivatives, the IBC image-dipole coefficients and
    // the real-space families that can come within r_c of the slab
    std::memset(&sh.img, 0, sizeof sh.img);
    sh.fam.clear();
    d.g1 = 1.0; d.cgam = 0.0; d.dg1t = d.dg1b = d.dcgt = d.dcgb = 0.0;
    for (int l = 1; l <= p.M; l++) {
        int a, b;
        exponents(l, +1, &a, &b);
        sh.img.ea_p[l - 1] = a; sh.img.eb_p[l - 1] = b;
        const double gpl = ipow(p.gamma_top, a) * ipow(p.gamma_bot, b);
        const double dpt = dmono(a, p.gamma_top, b, p.gamma_bot), dpb = dmono(b, p.gamma_bot, a, p.gamma_top);
        exponents(l, -1, &a, &b);
        sh.img.ea_m[l - 1] = a; sh.img.eb_m[l - 1] = b;
        const double gml = ipow(p.gamma_top, a) * ipow(p.gamma_bot, b);
        const double dmt = dmono(a, p.gamma_top, b, p.gamma_bot), dmb = dmono(b, p.gamma_bot, a, p.gamma_top);
        sh.img.gp[l - 1] = gpl; sh.img.gm[l - 1] = gml;
        const double sgn = (l % 2 == 0) ? 1.0 : -1.0;
        const double shp = 2.0 * ((l + 1) / 2) * p.H, shm = -2.0 * (l / 2) * p.H;
        d.g1 += sgn * (gpl + gml);
        d.cgam += shp * gpl + shm * gml;
        d.dg1t += sgn * (dpt + dmt); d.dg1b += sgn * (dpb + dmb);
        d.dcgt += shp * dpt + shm * dmt; d.dcgb += shp * dpb + shm * dmb;
        if ((l - 1) * p.H < p.r_c) {
            for (int side = 1; side >= -1; side -= 2) {
                Family f;
                if (l % 2) {   // reflection: target seen at sz = -1
                    f.sz = -1.0;
                    f.cz = side > 0 ? (l + 1) * p.H : -(l - 1) * p.H;
                    f.zsign = -1.0;
                } else {       // translation
                    f.sz = 1.0;
                    f.cz = side > 0 ? -l * p.H : l * p.H;
                    f.zsign = 1.0;
                }
                f.w = side > 0 ? gpl : gml;
                f.dwt = side > 0 ? dpt : dmt;
                f.dwb = side > 0 ? dpb : dmb;
                sh.fam.push_back(f);
            }
        }
    }
    if ((int)sh.fam.size() > kMaxFamilies)
        return fail(nullptr, RBE2D_E_INVAL, "too many image orders within r_c (H too small for r_c)");
    d.nfam = (int)sh.fam.size();

    // k-sampling tables and the FP32 phase split
    sh.cdf.assign(3, {});
    const double Ls[3] = {p.Lx, p.Ly, Lz};
    int nall = 0;
    for (int ax = 0; ax < 3; ax++) {
        axis_table(p.alpha, Ls[ax], &d.nmax[ax], sh.cdf[ax]);
        nall = std::max(nall, d.nmax[ax]);
    }
    int bits = 0;
    while ((1 << bits) <= nall) bits++;
    // fh keeps 22 - bits fraction bits: n fh then has at most 22 significant
    // bits for |n| < 2^bits, and nx fxh + ny fyh at most 23, so both are exact
    d.fh_bits = std::max(1, 22 - bits);
    d.scale_h = std::ldexp(1.0, d.fh_bits);
    if (p.precision == RBE2D_PREC_FP32_PHASE && bits > 20)
        return fail(nullptr, RBE2D_E_INVAL, "k-range too wide for FP32 phases (alpha L too large)");

    const bool fp32 = p.precision == RBE2D_PREC_FP32_PHASE;
    int ncx, ncy, ncz;
    d.snake = !fp32;
    if (fp32) scan_grid(p, d, &ncx, &ncy, &ncz);
    else tile_grid(p, d.nfam > 0, &ncx, &ncy, &ncz);
    d.ncx = ncx; d.ncy = ncy; d.ncz = ncz;
    d.hx = p.Lx / ncx; d.hy = p.Ly / ncy; d.hz = p.H / ncz;
    d.inv_hx = 1.0 / d.hx; d.inv_hy = 1.0 / d.hy; d.inv_hz = 1.0 / d.hz;
    d.inv_Lx = 1.0 / p.Lx; d.inv_Ly = 1.0 / p.Ly; d.inv_Lz = 1.0 / d.Lz;
    // fixed-point frame of the FP32 pair kernel.  z (and every transformed
    // target height within r_c of the slab) lies in [-zoff, zspan - zoff);
    // the span exceeds twice any candidate |dz| <= r_c + hz <= r_c + H.
    const double two32 = 4294967296.0;
    const double zspan = 2.0 * p.H + 4.0 * p.r_c;
    d.zoff = 0.5 * p.H + 2.0 * p.r_c;
    // candidates lie within r_c + hz of the target in z
    d.iso = p.Lx == p.Ly && 2.0 * (p.r_c + d.hz) * (1.0 + 1e-6) < p.Lx;
    d.fxs = two32 / p.Lx; d.fys = two32 / p.Ly; d.fzs = d.iso ? d.fxs : two32 / zspan;
    d.ux = (float)(p.Lx / two32); d.uy = (float)(p.Ly / two32);
    d.uz = d.iso ? d.ux : (float)(zspan / two32);
    d.rc2f = (float)(p.r_c * p.r_c);
    // below `near` the quantisation of the positions (one unit) would exceed
    // ~2^-22 of the distance: such pairs take exact FP64 displacements
    const double unit = d.iso ? p.Lx / two32 : std::max(std::max(p.Lx, p.Ly), zspan) / two32;
    const double near = unit * 4194304.0;
    d.near2f = (float)(near * near);
    d.ud = p.Lx / two32;
    d.u2 = (float)(d.ud * d.ud);
    d.rc2q = (float)(p.r_c * p.r_c * d.fxs * d.fxs);
    d.near2q = (float)(near * near * d.fxs * d.fxs);
    d.sig_top = d.sig_bot = 0.0;
    surface_setup(sh);
    return RBE2D_OK;
}

// Surface charges (reading R7): the uniform sheets sigma_bot on z = 0 and
// sigma_top on z = H, taken just inside the slab, and their images.  Every
// image of the bottom sheet below the slab (and the one at z = 0) pushes
// away from below, every image above pulls; the top sheet likewise.  For
// 0 < z < H this gives phi_s(z) = -Es z + Cs.  Net-charge term (reading R8):
// Gs, A1, A0 are the sums over the real charge and its images of w, w s c
// and w c^2 for image heights s z + c.  Index 0 is the value, 1 and 2 its
// derivatives by gamma_top and gamma_bot.
void surface_setup(SysHost &sh) {
    SysDesc &d = sh.d;
    const rbe2d_params &p = sh.p;
    for (int k = 0; k < 3; k++) { d.Es[k] = d.Cs[k] = d.A1[k] = d.A0[k] = 0.0; d.Gs[k] = k == 0 ? 1.0 : 0.0; }
    d.surf = (d.sig_top != 0.0 || d.sig_bot != 0.0) ? 1 : 0;
    // the real sheets: bottom at 0 (s = +1 for the ions above it), top at H (s = -1)
    d.Es[0] = 2.0 * kPi * (d.sig_bot - d.sig_top);
    d.Cs[0] = -2.0 * kPi * d.sig_top * d.H;          // -2 pi sigma_top |z - H| = 2 pi sigma_top (z - H)
    for (int l = 1; l <= p.M; l++) {
        int a, b;
        double wt[3], wb[3];   // weights (and gamma derivatives) of the + (above) and - (below) image
        exponents(l, +1, &a, &b);
        wt[0] = ipow(p.gamma_top, a) * ipow(p.gamma_bot, b);
        wt[1] = dmono(a, p.gamma_top, b, p.gamma_bot);
        wt[2] = dmono(b, p.gamma_bot, a, p.gamma_top);
        exponents(l, -1, &a, &b);
        wb[0] = ipow(p.gamma_top, a) * ipow(p.gamma_bot, b);
        wb[1] = dmono(a, p.gamma_top, b, p.gamma_bot);
        wb[2] = dmono(b, p.gamma_bot, a, p.gamma_top);
        const double s = (l % 2 == 0) ? 1.0 : -1.0;
        const double cp = 2.0 * ((l + 1) / 2) * p.H, cm = -2.0 * (l / 2) * p.H;
        // image heights of the bottom sheet (z = 0) and of the top sheet (z = H)
        const double bot_up = cp, bot_dn = cm, top_up = s * p.H + cp, top_dn = s * p.H + cm;
        for (int k = 0; k < 3; k++) {
            d.Gs[k] += wt[k] + wb[k];
            d.A1[k] += s * (wt[k] * cp + wb[k] * cm);
            d.A0[k] += wt[k] * cp * cp + wb[k] * cm * cm;
            // images above the slab pull (sign -1), below push (+1); the
            // potential -2 pi sigma w |z - z_w| = -2 pi sigma w sign (z - z_w)
            d.Es[k] += 2.0 * kPi * (d.sig_bot * (wb[k] - wt[k]) + d.sig_top * (wb[k] - wt[k]));
            d.Cs[k] += 2.0 * kPi * (d.sig_bot * (wb[k] * bot_dn - wt[k] * bot_up) +
                                    d.sig_top * (wb[k] * top_dn - wt[k] * top_up));
        }
    }
}

// Places buffers one after the other, 256-byte aligned, from `base` on (null:
// only adds up their sizes)
struct Carver {
    unsigned char *base = nullptr;
    size_t used = 0;
    template <typename T>
    void operator()(T **ptr, size_t count) {
        used = (used + 255) & ~(size_t)255;
        if (base) *ptr = (T *)(base + used);
        used += std::max<size_t>(count, 1) * sizeof(T);
    }
};

void prof_free(rbe2d_ctx *h) {
    Profiler &p = h->prof;
    for (int sl = 0; sl < RBE2D_PROF_SLOTS; sl++)
        for (int b = 0; b < 2; b++) {
            for (hipEvent_t e : p.ev[sl][b]) (void)hipEventDestroy(e);
            p.ev[sl][b].clear();
        }
    p.n = 0;
    for (int sl = 0; sl < RBE2D_PROF_SLOTS; sl++) p.used[sl] = 0;
}

void free_graph(rbe2d_ctx *h) {
    if (h->md_exec) (void)hipGraphExecDestroy(h->md_exec);
    if (h->md_graph) (void)hipGraphDestroy(h->md_graph);
    h->md_exec = nullptr;
    h->md_graph = nullptr;
    h->md_key.clear();
}

void free_all(rbe2d_ctx *h) {
    free_graph(h);
    prof_free(h);
    for (void *p : h->allocs) (void)hipFree(p);
    h->allocs.clear();
    if (h->kstage) (void)hipHostFree(h->kstage);
    if (h->lay_stage) (void)hipHostFree(h->lay_stage);
    if (h->kev) (void)hipEventDestroy(h->kev);
    if (h->lay_ev) (void)hipEventDestroy(h->lay_ev);
    if (h->fork_ev) (void)hipEventDestroy(h->fork_ev);
    if (h->join_ev) (void)hipEventDestroy(h->join_ev);
    if (h->cells_ev) (void)hipEventDestroy(h->cells_ev);
    if (h->side) (void)hipStreamDestroy(h->side);
}

// Every device workspace of a handle, in one fixed order: A(&ptr, count) is
// called once per buffer (count elements of *ptr's type).  The handle's
// capacities (n_sys, n_cap, cap_particles, cap_sorted, total_cells, P,
// precision) must be set.  own_kset: the handle holds its k-set (else the
// caller's device array is used in place).
template <typename Alloc>
void plan_workspace(rbe2d_ctx *h, size_t cdf_total, bool own_kset, Alloc &&A) {
    const int n = h->n_sys;
    const int cells = h->total_cells;
    const int64_t cap_blocks = h->cap_particles / kBlock;
    Workspace &w = h->w;
    A(&w.sys, n);
    A(&w.img, n);
    A(&w.fam, (size_t)n * kMaxFamilies);
    A(&w.cdf, cdf_total);
    A(&w.lay.off, n + 1); A(&w.lay.pbase, n + 1); A(&w.lay.bbase, n + 1);
    A(&w.lay.tbase, n + 1); A(&w.lay.sbase, n + 1);
    A(&w.p32, 2 * h->cap_particles);
    A(&w.p64, h->cap_particles);
    A(&w.bpart, 4 * cap_blocks);
    A(&w.scal, kScal * (size_t)n);
    if (own_kset) A(&w.kset, 3 * (size_t)n * h->P);
    A(&w.kn32, (size_t)n * h->P_pad);
    A(&w.kn64, (size_t)n * h->P_pad);
    double *sfp = nullptr;
    A(&sfp, (size_t)cap_blocks * h->P_pad * 4);
    w.sfpart = sfp;
    A(&w.krec, (size_t)n * h->P * kKRec);
    A(&w.kf32, 3 * (size_t)n * h->P);
    A(&w.kf64, kKF64 * (size_t)n * h->P);
    A(&w.fpart, h->P > kLongP ? std::min<int64_t>(kMaxForceRows * cap_blocks, kMaxRowBlocks) * kBlock : 0);
    const int64_t nc = std::max<int64_t>(h->n_cap, 1);
    A(&w.cell, nc); A(&w.slot, nc); A(&w.tmp, nc);
    A(&w.count, cells); A(&w.start, cells + 1); A(&w.scanbuf, cells / 1024 + 2);
    A(&w.sorted, h->cap_sorted); A(&w.sidx, h->cap_sorted);
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    // the FP32 records get one wave of padding: the pair kernel reads the first
    // record of an empty run, which may start at the end of the array
    if (fp32) { A(&w.src16, h->cap_sorted + kWave); A(&w.scell, h->cap_sorted); }
    A(&w.freal, nc); A(&w.fshort, h->one_stream ? 0 : nc);   // (the call without a handle has no MD)
    A(&w.rpart, 3 * (h->cap_sorted / kWave));
    // FP32 pair kernel: the split is only used when there are too few targets
    // to fill the chip
    h->split_cap = fp32 ? std::min<int64_t>(nc, 1 << 18) : 0;
    const int64_t fam_cap = fp32 ? std::min<int64_t>(nc, kFamilySplitMax) : 0;
    int64_t parts = std::max(kMaxRealSplit * h->split_cap, kMaxRealSplit * kMaxFamilySplit * fam_cap);
    int64_t wparts = kMaxRealSplit * kMaxFamilySplit * (h->cap_sorted / kWave);
    // FP64: as many parts as there are blocks, of 64 targets each at most
    if (!fp32) parts = (wparts = kTileBlocks) * kWave;
    A(&w.freal_s, parts);
    A(&w.rpart_s, 3 * wparts);
    A(&w.spart, 2 * (h->cap_sorted / kWave));
    A(&w.err, 4);
    A(&w.step, 1);
}

// A handle over n systems: every system is set up and the workspaces are
// sized for the sum of their n_max.
rbe2d_status create_handle(int n, const rbe2d_params *ps, bool batch, rbe2d_handle *out) {
    if (!out) return fail(nullptr, RBE2D_E_INVAL, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > 65536) return fail(nullptr, RBE2D_E_INVAL, "n_sys must be in [1, 65536]");
    if (!ps) return fail(nullptr, RBE2D_E_INVAL, "params is NULL");
    rbe2d_ctx *h = new (std::nothrow) rbe2d_ctx();
    if (!h) return fail(nullptr, RBE2D_E_NOMEM, "host allocation failed");
    h->n_sys = n;
    h->batch = batch;
    h->sys.resize(n);
    int64_t n_cap = 0, cap_p = 0, cap_s = 0;
    int cells = 0;
    size_t cdf_total = 0;
    for (int r = 0; r < n; r++) {
        rbe2d_status st = setup_system(&ps[r], h->sys[r]);
        if (st) {
            delete h;
            if (n > 1) g_create_error = "system " + std::to_string(r) + ": " + g_create_error;
            return st;
        }
        const rbe2d_params &p = h->sys[r].p;
        if (r > 0 && (p.P != h->sys[0].p.P || p.precision != h->sys[0].p.precision)) {
            delete h;
            return fail(nullptr, RBE2D_E_INVAL, "all systems of a batch need the same P and precision");
        }
        SysDesc &d = h->sys[r].d;
        d.cbase = cells;
        cells += d.ncx * d.ncy * d.ncz;
        h->max_cells = std::max(h->max_cells, d.ncx * d.ncy * d.ncz);
        for (int ax = 0; ax < 3; ax++) {
            d.cdf_off[ax] = (int)cdf_total;
            cdf_total += h->sys[r].cdf[ax].size();
        }
        n_cap += p.n_max;
        cap_p += (p.n_max + kTileMax - 1) / kTileMax * kTileMax;
        cap_s += (p.n_max + kWave - 1) / kWave * kWave;
    }
    if (n_cap > INT32_MAX - kTileMax || cap_p > INT32_MAX / 2 || cells > INT32_MAX / 2) {
        delete h;
        return fail(nullptr, RBE2D_E_INVAL, "total particle or cell capacity exceeds 2^30");
    }
    h->precision = h->sys[0].p.precision;
    h->iso = true;
    for (int r = 0; r < n; r++) h->iso = h->iso && h->sys[r].d.iso;
    h->P = h->sys[0].p.P;
    h->P_pad = (h->P + kPPad - 1) / kPPad * kPPad;
    h->n_cap = n_cap;
    h->cap_particles = std::max<int64_t>(cap_p, kTileMax);
    h->cap_sorted = std::max<int64_t>(cap_s, kWave);
    h->total_cells = cells;
    h->split_blocks = 4096;
    (void)hipGetDevice(&h->device);

    // all workspaces in one allocation, cleared at once (each of the 40 apart
    // took two runtime calls)
    Carver sizes, ws;
    plan_workspace(h, cdf_total, true, sizes);
    hipError_t e = hipMalloc((void **)&ws.base, sizes.used);
    if (e == hipSuccess) {
        h->allocs.push_back(ws.base);
        e = hipMemset(ws.base, 0, sizes.used);
        plan_workspace(h, cdf_total, true, ws);
    }
    Workspace &w = h->w;
    std::vector<SysDesc> descs(n);
    std::vector<ImgTable> imgs(n);
    std::vector<Family> fams((size_t)n * kMaxFamilies);
    std::vector<double> cdf(cdf_total);
    for (int r = 0; r < n; r++) {
        descs[r] = h->sys[r].d;
        imgs[r] = h->sys[r].img;
        std::copy(h->sys[r].fam.begin(), h->sys[r].fam.end(), fams.begin() + (size_t)r * kMaxFamilies);
        for (int ax = 0; ax < 3; ax++)
            std::copy(h->sys[r].cdf[ax].begin(), h->sys[r].cdf[ax].end(), cdf.begin() + descs[r].cdf_off[ax]);
    }
    if (e == hipSuccess) e = hipMemcpy(w.sys, descs.data(), n * sizeof(SysDesc), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(w.img, imgs.data(), n * sizeof(ImgTable), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(w.fam, fams.data(), fams.size() * sizeof(Family), hipMemcpyHostToDevice);
    if (e == hipSuccess && cdf_total)
        e = hipMemcpy(w.cdf, cdf.data(), cdf_total * sizeof(double), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipHostMalloc((void **)&h->kstage, 3 * sizeof(int32_t) * n * h->P, hipHostMallocDefault);
    if (e == hipSuccess) e = hipHostMalloc((void **)&h->lay_stage, 5 * sizeof(int) * (n + 1), hipHostMallocDefault);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&h->kev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&h->lay_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&h->fork_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&h->join_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&h->cells_ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        const bool oom = e == hipErrorOutOfMemory;
        free_all(h);
        delete h;
        return fail(nullptr, oom ? RBE2D_E_NOMEM : RBE2D_E_HIP, "workspace setup failed: %s",
                    hipGetErrorString(e));
    }
    *out = h;
    return RBE2D_OK;
}

// Particle layout of all systems for the given counts into lay (5 (n_sys +
// 1) ints: off, pbase, bbase, tbase, sbase) and the handle's launch sizes.
rbe2d_status compute_layout(rbe2d_ctx *h, const int64_t *counts, int *lay) {
    const int n = h->n_sys;
    int64_t total = 0;
    for (int r = 0; r < n; r++) {
        if (counts[r] < 0 || counts[r] > h->sys[r].p.n_max)
            return fail(h, RBE2D_E_INVAL, "system %d: N = %lld outside [0, n_max = %lld]", r,
                        (long long)counts[r], (long long)h->sys[r].p.n_max);
        total += counts[r];
    }
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    const int nkc = h->P_pad / (fp32 ? kKChunk32 : kKChunk64);
    h->tuned_now = !h->tune.counts.empty() && std::equal(counts, counts + n, h->tune.counts.begin());
    int per;
    if (h->force_per) {
        per = h->force_per;
    } else if (h->tuned_now && h->tune.per) {
        per = h->tune.per;
    } else {
        // tile size: enough tiles to fill the chip, padding under ~10% of the particles
        per = choose_tile(total, nkc);
        for (; per > 1; per >>= 1) {
            int64_t padded = 0;
            const int64_t tile = (int64_t)kBlock * per;
            for (int r = 0; r < n; r++) padded += (counts[r] + tile - 1) / tile * tile;
            if (padded <= total + total / 10 + tile) break;
        }
    }
    const int tile = kBlock * per;
    std::fill(lay, lay + 5 * (n + 1), 0);
    int *off = lay, *pb = off + (n + 1), *bb = pb + (n + 1), *tb = bb + (n + 1), *sb = tb + (n + 1);
    for (int r = 0; r < n; r++) {
        off[r + 1] = off[r] + (int)counts[r];
        pb[r + 1] = pb[r] + (int)((counts[r] + tile - 1) / tile * tile);
        sb[r + 1] = sb[r] + (int)((counts[r] + kWave - 1) / kWave * kWave);
    }
    for (int r = 0; r <= n; r++) { bb[r] = pb[r] / kBlock; tb[r] = pb[r] / tile; }
    h->per = per;
    h->n_total = total;
    h->max_n = n > 0 ? (int)*std::max_element(counts, counts + n) : 0;
    h->n_blocks = bb[n];
    h->n_tiles = tb[n];
    h->n_swaves = sb[n] / kWave;
    return RBE2D_OK;
}

// Every call counts the particles per cell from zero, and its cell list clears
// the counts.  Counts of a call that failed in between are cleared at its end
// (CountGuard: replays of a captured call count from zero as well), or, where
// that launch fails too, when the next call begins.
hipError_t clear_counts(rbe2d_ctx *h, hipStream_t s) {
    if (!h->cells_counted) return hipSuccess;
    (void)hipGetLastError();   // (the failure that left them, reported by its call)
    const hipError_t e = launch_fill(h->w.count, (int64_t)h->total_cells * 4, s);
    if (e == hipSuccess) h->cells_counted = false;
    return e;
}
struct CountGuard {
    rbe2d_ctx *h;
    hipStream_t s;
    ~CountGuard() { (void)clear_counts(h, s); }
};

// Particle layout of all systems for the given counts; uploaded (through
// pinned staging, ordered on the stream) only when it changes.
rbe2d_status set_layout(rbe2d_ctx *h, const int64_t *counts, hipStream_t s) {
    const int n = h->n_sys;
    h->calls++;
    std::vector<int> lay(5 * (n + 1), 0);
    rbe2d_status st = compute_layout(h, counts, lay.data());
    if (st) return st;
    RBE2D_TRY(h, clear_counts(h, s), "count clear");
    if (h->lay_valid && lay == h->lay_host) return RBE2D_OK;
    if (h->lay_ev_pending) RBE2D_TRY(h, hipEventSynchronize(h->lay_ev), "layout wait");
    std::memcpy(h->lay_stage, lay.data(), lay.size() * sizeof(int));
    int *dst[5] = {h->w.lay.off, h->w.lay.pbase, h->w.lay.bbase, h->w.lay.tbase, h->w.lay.sbase};
    for (int k = 0; k < 5; k++)
        RBE2D_TRY(h, hipMemcpyAsync(dst[k], h->lay_stage + k * (n + 1), (n + 1) * sizeof(int),
                                    hipMemcpyHostToDevice, s), "layout upload");
    RBE2D_TRY(h, hipEventRecord(h->lay_ev, s), "layout event");
    h->lay_ev_pending = true;
    h->neighbours = 0.0;
    for (int r = 0; r < n && h->n_total > 0; r++) {
        const rbe2d_params &p = h->sys[r].p;
        const double c = (double)counts[r], ball = 4.0 / 3.0 * kPi * p.r_c * p.r_c * p.r_c;
        h->neighbours += c * c / h->n_total / (p.Lx * p.Ly * p.H) *
                         (h->sys[r].d.nfam > 0 ? ball : std::min(ball, kPi * p.r_c * p.r_c * p.H));
    }
    h->lay_host = lay;
    h->lay_valid = true;
    return RBE2D_OK;
}

rbe2d_status layout_from_offsets(rbe2d_ctx *h, const int64_t *offsets, hipStream_t s) {
    if (!offsets) return fail(h, RBE2D_E_INVAL, "offsets is NULL");
    if (offsets[0] != 0) return fail(h, RBE2D_E_INVAL, "offsets[0] must be 0");
    std::vector<int64_t> counts(h->n_sys);
    for (int r = 0; r < h->n_sys; r++) {
        counts[r] = offsets[r + 1] - offsets[r];
        if (counts[r] < 0) return fail(h, RBE2D_E_INVAL, "offsets must be nondecreasing");
    }
    return set_layout(h, counts.data(), s);
}

rbe2d_status check_arrays(rbe2d_ctx *h, const double *pos, const double *q) {
    if (!h->kset_valid) return fail(h, RBE2D_E_STATE, "no k-set: call rbe2d_set_kset or rbe2d_sample_kset");
    if (h->n_total > 0 && (!pos || !q)) return fail(h, RBE2D_E_INVAL, "pos or q is NULL");
    return RBE2D_OK;
}

// One stream for the whole call?  Two let the k-space chain and the pair
// kernel share the chip, but cost four event calls (10 us each on the host)
// and the waits between streams; on one, the k-space work rides along with the
// real-space launches.  us per force call on one stream | two: 1000 ions FP64
// 62 | 70, 4000 FP32 71 | 79, 16000 FP64 76 | 87, 24000 FP32 86 | 88 and
// 122 | 124, 48000 FP32 122 | 121 and 185 | 172, 90000 FP64 203 | 215 and
// 256 | 259.  Energy and gradient, whose caller waits for each: 4000 ions
// 173 | 232, 90000 FP64 380 | 454, 90000 FP32 380 | 391.  With many wave vectors
// (of all systems) the assembly fills the chip by itself and gains by the pair
// kernel beside it: FP64, 4096 slabs of 16 ions with 32 each 368 | 339, 16 slabs
// of 500 with 4000 287 | 275, 64 of 300 with 500 167 | 162, but 1024 of 16 with
// 32 126 | 145.  (A structure-factor launch of its own deals
// whole tiles to the XCDs and wants two for each at least: 500 ions with 65536
// wave vectors 968 | 2447, energy of 40000 with 40000 1808 | 2588.)
constexpr int64_t kOneStreamForces32 = 24576, kOneStream = 98304, kOneStreamItems = 32768;
bool on_one_stream(const rbe2d_ctx *h, bool energy) {
    return h->one_stream ||
           (h->n_total <= (!energy && h->precision == RBE2D_PREC_FP32_PHASE ? kOneStreamForces32 : kOneStream) &&
            ((int64_t)h->n_sys * h->P <= kOneStreamItems || h->n_tiles < 16));
}

// On one stream the structure factors and the assembly ride along with the
// real-space launches (not while the launches are timed class by class)
bool rides_along(const rbe2d_ctx *h, bool one_stream) { return one_stream && h->n_total > 0 && h->prof.n == 0; }

// A pair kernel whose waves are all on the chip at once lasts as long as the
// latest of them: the structure factors then start after the cell list, beside
// the pair kernel, and not on the chip before it.  us per call with the fork
// before | after the cell list: energy and gradient of 150000 ions FP32 631 |
// 557, FP64 693 | 533; forces of 150000 ions FP64 450 | 377, FP32 484 | 447 and
// 281 | 258, of 250000 FP32 662 | 511; but of 100000 FP32, where the pair work is
// split over more waves, 284 | 270 and 197 | 214.  With FP32 phases it takes more
// pairs than the k-space chain has wave vectors to last longer than it, per ion
// 0.6 neighbours for each (forces: two passes) or 0.3 (energies: one).  Forces of
// 200000 ions, neighbours for each wave vector: 0.17 139 | 161, 0.27 294 | 310,
// 0.44 170 | 185, 0.64 456 | 423, 0.70 206 | 207, 1.05 251 | 242; energies of
// 200000, 0.11 189 | 206, 0.17 129 | 145, 0.27 271 | 255, 0.44 172 | 170, 0.70
// 208 | 195.  Where the pair kernel leaves half of the chip, up to 2304 waves,
// forces take less: 140000 ions, 0.17 110 | 128, 0.27 248 | 225.
bool pairs_first(const rbe2d_ctx *h, bool energy) {
    if (h->n_swaves > 4096) return false;
    if (h->precision != RBE2D_PREC_FP32_PHASE) return true;
    return (energy || h->n_swaves > 2048) && h->neighbours >= (energy ? 0.3 : h->n_swaves <= 2304 ? 0.25 : 0.6) * h->P;
}

// `to` waits for what `from` has been given so far
rbe2d_status stream_wait(rbe2d_ctx *h, hipStream_t to, hipStream_t from, hipEvent_t ev) {
    RBE2D_TRY(h, hipEventRecord(ev, from), "stream event");
    RBE2D_TRY(h, hipStreamWaitEvent(to, ev, 0), "stream wait");
    return RBE2D_OK;
}

// prep + structure factors + real space: everything the outputs depend on.
// With both halves requested, the k-space chain (structure factors, per-k
// assembly) runs on the side stream while the cell list and the pair kernel
// run on `s`; `s` waits for both.  The cell build is latency- and
// atomic-bound and the pair kernel latency-limited, so the VALU-bound
// structure-factor pass fills their idle issue slots.  The fork and join are
// events, so the pattern is also captured into graphs.
rbe2d_status run_common(rbe2d_ctx *h, const double *pos, const double *q, uint32_t flags, bool want_dg,
                        hipStream_t s) {
    const bool kside = (flags & (RBE2D_KSPACE | RBE2D_IBC)) != 0;
    const bool real = (flags & RBE2D_REAL) != 0;
    // with k-space the assembly launch computes the IBC scalars
    const bool sc_asm = (flags & RBE2D_KSPACE) != 0;
    if (kside) RBE2D_TRY(h, launch_prep(h, pos, q, s, !sc_asm, real), "prep launch");
    const bool two = sc_asm && real && h->n_total > 0 && !on_one_stream(h, true);
    const bool late = two && pairs_first(h, true);
    if (two && !late) {
        rbe2d_status st = stream_wait(h, h->side, s, h->fork_ev);
        if (st) return st;
    }
    // real space is enqueued first: its cell list starts ahead of the structure factors
    const bool ride = rides_along(h, sc_asm && real && !two);
    if (real)
        RBE2D_TRY(h, launch_real(h, pos, q, want_dg, s, ride, late ? h->fork_ev : nullptr),
                  "real-space launch");
    if (late) RBE2D_TRY(h, hipStreamWaitEvent(h->side, h->fork_ev, 0), "stream wait");
    if (sc_asm && !ride) RBE2D_TRY(h, launch_kcoef_sf(h, two ? h->side : s, true, want_dg), "structure-factor launch");
    return two ? stream_wait(h, s, h->side, h->join_ev) : RBE2D_OK;
}

// What compute_forces does besides the forces: the closing half kick
// v += dt/2 F of an MD step (vel), the MD's short-range forces (mx), the
// energies and a copy of the error word.
struct ForceJob {
    double *vel = nullptr;
    double dt = 0.0;
    const MdExtra *mx = nullptr;
    double *energy = nullptr;
    int32_t *err_out = nullptr;
    bool prepared = false;        // an MD pass has prepared particles, cells and k-set (parts: all)
    long long *step = nullptr;    // MD step counter to advance once the k-set's step is over
};

// Forces of `parts` into F (added to F with `accumulate`).  With real space
// and k-space/IBC both requested, the whole k-space chain including its force
// scatter runs on the side stream (writing F) while the cell list, the pair
// kernel and the short-range kernel run on `s`; after the join one pass adds
// their forces, with the half kick and the energies as part of it.  On one
// stream the force scatter comes last and does all of that.
rbe2d_status compute_forces(rbe2d_ctx *h, const double *pos, const double *q, double *F, uint32_t parts,
                            bool accumulate, const ForceJob &job, hipStream_t s) {
    const bool kside = (parts & (RBE2D_KSPACE | RBE2D_IBC)) != 0, real = (parts & RBE2D_REAL) != 0;
    const bool sc_asm = (parts & RBE2D_KSPACE) != 0;
    // (MD steps, captured or not: two streams; captured, 2000 ions take 63 us
    // per Langevin step in FP64 against 74, 75 against 77 in FP32)
    const bool two = kside && real && h->n_total > 0 && (job.prepared ? !h->one_stream : !on_one_stream(h, false));
    if (kside && !job.prepared) RBE2D_TRY(h, launch_prep(h, pos, q, s, !sc_asm, real), "prep launch");
    hipStream_t ks = two ? h->side : s;
    const bool late = two && !job.prepared && pairs_first(h, false);
    if (two && !late) {
        rbe2d_status st = stream_wait(h, ks, s, h->fork_ev);
        if (st) return st;
    }
    // real space first: its latency-bound cell list then starts ahead of the
    // structure factors (also in a captured graph, whose nodes follow this order)
    const bool ride = rides_along(h, sc_asm && real && !two);
    // (an MD step: two streams)  The short-range kernel needs the cell list
    // only: after the k-space chain on the side stream, beside the pair kernel,
    // or, where that chain is the longer one, after the pair kernel.
    const bool shortr = two && job.mx;
    const bool short_side = h->precision != RBE2D_PREC_FP32_PHASE || h->n_total <= kShortTiles32;
    if (real)
        RBE2D_TRY(h, launch_real(h, pos, q, false, s, ride, late ? h->fork_ev : shortr && short_side ? h->cells_ev : nullptr),
                  "real-space launch");
    if (late) RBE2D_TRY(h, hipStreamWaitEvent(ks, h->fork_ev, 0), "stream wait");
    if (shortr && !short_side)
        RBE2D_TRY(h, launch_short(h, *job.mx, nullptr, nullptr, s), "short-range launch");
    if (sc_asm && !ride) RBE2D_TRY(h, launch_kcoef_sf(h, ks, true, false, job.step), "structure-factor launch");
    ForceExtra x;
    if (!two) {
        x.energy = job.energy; x.err_out = job.err_out;
    }
    RBE2D_TRY(h, launch_kforce(h, pos, q, F, nullptr, two ? parts & ~(uint32_t)RBE2D_REAL : parts, accumulate, false,
                               real && !two, nullptr, ks, x), "force launch");
    if (two) {
        if (shortr && short_side) {
            RBE2D_TRY(h, hipStreamWaitEvent(ks, h->cells_ev, 0), "stream wait");
            RBE2D_TRY(h, launch_short(h, *job.mx, nullptr, nullptr, ks), "short-range launch");
        }
        rbe2d_status st = stream_wait(h, s, ks, h->join_ev);
        if (st) return st;
        RBE2D_TRY(h, launch_add_real(h, F, job.vel, 0.5 * job.dt, s, job.energy, parts), "real-space add");
        if (job.err_out) RBE2D_TRY(h, launch_copy_err(h, job.err_out, s), "error word");
    }
    if (h->n_total == 0) {   // (no force pass)
        if (job.energy) RBE2D_TRY(h, launch_energy(h, job.energy, parts, nullptr, nullptr, s), "energy launch");
        if (job.err_out) RBE2D_TRY(h, launch_copy_err(h, job.err_out, s), "error word");
    }
    return RBE2D_OK;
}

rbe2d_status run_forces(rbe2d_ctx *h, const double *pos, const double *q, double *F, double *energy,
                        uint32_t flags, hipStream_t s) {
    const CountGuard guard{h, s};
    if (flags & ~(uint32_t)(RBE2D_ALL | RBE2D_ACCUMULATE)) return fail(h, RBE2D_E_INVAL, "unknown flags");
    rbe2d_status st = check_arrays(h, pos, q);
    if (st) return st;
    if (h->n_total > 0 && !F) return fail(h, RBE2D_E_INVAL, "F is NULL");
    ForceJob job;
    job.energy = energy;
    return compute_forces(h, pos, q, F, flags & RBE2D_ALL, (flags & RBE2D_ACCUMULATE) != 0, job, s);
}

rbe2d_status md_extra(rbe2d_ctx *h, const rbe2d_md_params *mp, double dt, MdExtra *mx) {
    if (!mp) return fail(h, RBE2D_E_INVAL, "md params are NULL");
    const double vals[] = {mp->gamma, mp->kT, mp->sigma, mp->eps, mp->sigma_wall, mp->eps_wall, mp->wall_margin};
    for (double v : vals)
        if (!std::isfinite(v)) return fail(h, RBE2D_E_INVAL, "non-finite md parameter");
    if (mp->gamma < 0 || mp->kT < 0 || mp->eps < 0 || mp->eps_wall < 0)
        return fail(h, RBE2D_E_INVAL, "gamma, kT, eps, eps_wall must be >= 0");
    if ((mp->eps > 0 && !(mp->sigma > 0)) || (mp->eps_wall > 0 && !(mp->sigma_wall > 0)))
        return fail(h, RBE2D_E_INVAL, "sigma, sigma_wall must be > 0 where eps, eps_wall are");
    double hmin = h->sys[0].p.H;
    for (const SysHost &sh : h->sys) hmin = std::min(hmin, sh.p.H);
    if (!(mp->wall_margin > 0 && 2 * mp->wall_margin < hmin))
        return fail(h, RBE2D_E_INVAL, "need 0 < wall_margin < H/2");
    const double rlj = std::pow(2.0, 1.0 / 6.0) * mp->sigma;
    for (const SysHost &sh : h->sys)
        if (mp->eps > 0 && 2 * rlj > std::min(sh.p.Lx, sh.p.Ly))
            return fail(h, RBE2D_E_INVAL, "ion-ion LJ cutoff exceeds half the box");
    mx->c1 = std::exp(-mp->gamma * dt);
    mx->c2 = std::sqrt((1.0 - mx->c1 * mx->c1) * mp->kT);
    mx->sig2 = mp->sigma * mp->sigma;
    mx->eps = mp->eps;
    mx->rc2 = rlj * rlj;
    mx->sigw2 = mp->sigma_wall * mp->sigma_wall;
    mx->epsw = mp->eps_wall;
    mx->hcut = std::pow(2.0, 1.0 / 6.0) * mp->sigma_wall;
    mx->margin = mp->wall_margin;
    return RBE2D_OK;
}

// one BAOAB step of mx with its short-range forces (without mx: a step of an
// empty layout, which only draws its k-set); the k-set and the thermostat
// noise use the device step counter when dev_step is set (graph replays),
// else stream id `step`
rbe2d_status md_step(rbe2d_ctx *h, double *pos, double *vel, const double *q, double *F, double dt,
                     double zlo, double zhi_from_top, uint64_t seed, int64_t step, bool dev_step,
                     const MdExtra *mx, hipStream_t s) {
    const uint64_t sbase = (uint64_t)step * (uint64_t)h->n_sys;
    if (mx) zlo = zhi_from_top = mx->margin;
    RBE2D_TRY(h, launch_prep_md(h, mx ? 3 : 1, pos, vel, F, q, dt, zlo, zhi_from_top, mx, seed, sbase,
                                dev_step ? h->w.step : nullptr, s), "md drift");
    ForceJob job;
    job.vel = vel; job.dt = dt; job.prepared = true;
    job.mx = mx && mx->short_on() ? mx : nullptr;
    job.step = dev_step ? h->w.step : nullptr;
    return compute_forces(h, pos, q, F, RBE2D_ALL, false, job, s);
}

// Force evaluation and closing kick of one plain velocity-Verlet step at
// the current positions (whose k-set is drawn, with its k-vector table, and
// whose k-space particle records and IBC block sums the preceding MD pass
// wrote).  The k-space chain (structure factors, assembly with the IBC
// scalars, force scatter) runs on the side stream, real space on s (also for
// small systems: 500 ions 55 us per step FP32, 63 on one stream as in
// compute_forces; 16000 ions 92 and 104).  After
// the forces, either the closing half kick (last step of the run) or one
// pass with the closing and next opening half kicks, the next drift, the next
// records and the next k-set (device step counter: advanced by the assembly).
rbe2d_status vv_unit(rbe2d_ctx *h, double *pos, double *vel, const double *q, double *F, double dt, double zlo,
                     double zhi_from_top, uint64_t seed, int64_t step, bool dev_step, bool last, hipStream_t s) {
    long long *counter = dev_step ? h->w.step : nullptr;
    hipStream_t ks = h->side;
    rbe2d_status st = stream_wait(h, ks, s, h->fork_ev);
    if (st) return st;
    // real space first: its latency-bound cell list then starts ahead of the
    // structure factors (also in a captured graph, whose nodes follow this order)
    RBE2D_TRY(h, launch_real(h, pos, q, false, s), "real-space launch");
    RBE2D_TRY(h, launch_kcoef_sf(h, ks, true, false, counter), "structure-factor launch");
    RBE2D_TRY(h, launch_kforce(h, pos, q, F, nullptr, RBE2D_KSPACE | RBE2D_IBC, false, false, false, nullptr, ks),
              "force launch");
    st = stream_wait(h, s, ks, h->join_ev);
    if (st) return st;
    if (!last)
        RBE2D_TRY(h, launch_prep_md(h, 2, pos, vel, F, q, dt, zlo, zhi_from_top, nullptr, seed,
                                    (uint64_t)(step + 1) * (uint64_t)h->n_sys, counter, s),
                  "md leapfrog");
    else
        RBE2D_TRY(h, launch_add_real(h, F, vel, 0.5 * dt, s), "real-space add");
    return RBE2D_OK;
}

// plain velocity Verlet (no thermostat, no short-range forces) over n steps:
// the opening kick and drift with the caller's F and the first k-draw, then
// n force evaluations chained by fused kicks; with use_graph the middle ones
// are replays of one captured unit
rbe2d_status vv_run(rbe2d_ctx *h, double *pos, double *vel, const double *q, double *F, double dt, double zlo,
                    double zhi_from_top, uint64_t seed, int64_t step0, int32_t n_steps, bool use_graph,
                    hipStream_t s) {
    RBE2D_TRY(h, launch_prep_md(h, 1, pos, vel, F, q, dt, zlo, zhi_from_top, nullptr, seed,
                                (uint64_t)step0 * (uint64_t)h->n_sys, nullptr, s), "md drift");
    int32_t it = 0;
    if (use_graph) {
        auto bits = [](double x) { uint64_t u; std::memcpy(&u, &x, 8); return u; };
        std::vector<uint64_t> key = {1, (uint64_t)(uintptr_t)pos, (uint64_t)(uintptr_t)vel, (uint64_t)(uintptr_t)q,
                                     (uint64_t)(uintptr_t)F, bits(dt), bits(zlo), bits(zhi_from_top), seed,
                                     (uint64_t)h->per};
        key.insert(key.end(), h->lay_host.begin(), h->lay_host.end());
        if (!h->md_exec || key != h->md_key) {
            free_graph(h);
            hipStream_t cs;
            RBE2D_TRY(h, hipStreamCreateWithFlags(&cs, hipStreamNonBlocking), "capture stream");
            const int prof_n = h->prof.n;
            h->prof.n = 0;   // no profiling events inside the graph
            // a captured unit starts from counted cells and ends by counting
            // them for the next one; a failed capture leaves the state as it was
            const bool counted0 = h->cells_counted;
            hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
            rbe2d_status st = RBE2D_OK;
            if (e == hipSuccess) {
                st = vv_unit(h, pos, vel, q, F, dt, zlo, zhi_from_top, seed, 0, true, false, cs);
                hipGraph_t g = nullptr;
                const hipError_t e2 = hipStreamEndCapture(cs, &g);
                if (st == RBE2D_OK && e2 != hipSuccess) st = hipfail(h, e2, "end capture");
                if (st == RBE2D_OK) {
                    h->md_graph = g;
                    const hipError_t e3 = hipGraphInstantiate(&h->md_exec, g, nullptr, nullptr, 0);
                    if (e3 != hipSuccess) st = hipfail(h, e3, "graph instantiate");
                } else if (g) {
                    (void)hipGraphDestroy(g);
                }
            } else {
                st = hipfail(h, e, "begin capture");
            }
            h->prof.n = prof_n;
            (void)hipStreamDestroy(cs);
            h->cells_counted = counted0;
            if (st) { free_graph(h); return st; }
            h->md_key = key;
        }
        RBE2D_TRY(h, launch_set_step(h, step0, s), "md step counter");
        for (; it < n_steps - 1; it++) RBE2D_TRY(h, hipGraphLaunch(h->md_exec, s), "graph launch");
    }
    for (; it < n_steps; it++) {
        rbe2d_status st = vv_unit(h, pos, vel, q, F, dt, zlo, zhi_from_top, seed, step0 + it, false,
                                  it == n_steps - 1, s);
        if (st) return st;
    }
    return RBE2D_OK;
}

// n_steps MD steps, eager or as replays of one captured step
rbe2d_status md_run(rbe2d_ctx *h, double *pos, double *vel, const double *q, double *F, double dt, double zlo,
                    double zhi_from_top, uint64_t seed, int64_t step0, int32_t n_steps, bool use_graph,
                    const MdExtra *mx, hipStream_t s) {
    if (n_steps <= 0) return RBE2D_OK;
    const CountGuard guard{h, s};
    h->kset_valid = true;
    if (!mx && h->n_total > 0)
        return vv_run(h, pos, vel, q, F, dt, zlo, zhi_from_top, seed, step0, n_steps, use_graph, s);
    if (!use_graph) {
        for (int32_t it = 0; it < n_steps; it++) {
            rbe2d_status st = md_step(h, pos, vel, q, F, dt, zlo, zhi_from_top, seed, step0 + it, false, mx, s);
            if (st) return st;
        }
        return RBE2D_OK;
    }
    // a captured step is valid for these arguments and this layout only
    auto bits = [](double x) { uint64_t u; std::memcpy(&u, &x, 8); return u; };
    std::vector<uint64_t> key = {(uint64_t)(uintptr_t)pos, (uint64_t)(uintptr_t)vel, (uint64_t)(uintptr_t)q,
                                 (uint64_t)(uintptr_t)F, bits(dt), bits(zlo), bits(zhi_from_top), seed,
                                 (uint64_t)h->per};
    if (mx)
        for (double v : {mx->c1, mx->c2, mx->sig2, mx->eps, mx->rc2, mx->sigw2, mx->epsw, mx->hcut, mx->margin})
            key.push_back(bits(v));
    key.insert(key.end(), h->lay_host.begin(), h->lay_host.end());
    if (!h->md_exec || key != h->md_key) {
        free_graph(h);
        hipStream_t cs;
        RBE2D_TRY(h, hipStreamCreateWithFlags(&cs, hipStreamNonBlocking), "capture stream");
        const int prof_n = h->prof.n;
        h->prof.n = 0;   // no profiling events inside the graph
        const bool counted0 = h->cells_counted;   // (a failed capture has counted nothing)
        hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
        rbe2d_status st = RBE2D_OK;
        if (e == hipSuccess) {
            st = md_step(h, pos, vel, q, F, dt, zlo, zhi_from_top, seed, 0, true, mx, cs);
            hipGraph_t g = nullptr;
            const hipError_t e2 = hipStreamEndCapture(cs, &g);
            if (st == RBE2D_OK && e2 != hipSuccess) st = hipfail(h, e2, "end capture");
            if (st == RBE2D_OK) {
                h->md_graph = g;
                const hipError_t e3 = hipGraphInstantiate(&h->md_exec, g, nullptr, nullptr, 0);
                if (e3 != hipSuccess) st = hipfail(h, e3, "graph instantiate");
            } else if (g) {
                (void)hipGraphDestroy(g);
            }
        } else {
            st = hipfail(h, e, "begin capture");
        }
        h->prof.n = prof_n;
        (void)hipStreamDestroy(cs);
        h->cells_counted = counted0;
        if (st) { free_graph(h); return st; }
        h->md_key = key;
    }
    RBE2D_TRY(h, launch_set_step(h, step0, s), "md step counter");
    for (int32_t it = 0; it < n_steps; it++) RBE2D_TRY(h, hipGraphLaunch(h->md_exec, s), "graph launch");
    return RBE2D_OK;
}

// ---------------------------------------------------------------------------
// The evaluation without a handle (rbe2d_forces_noalloc): every workspace is
// carved from one file-scope device array, so a call allocates no device or
// pinned memory and creates no stream or event.
// ---------------------------------------------------------------------------

constexpr int64_t kStaticMaxN = 32768;     // largest n_max of the static path
constexpr int kStaticMaxP = 1024;          // largest P of the static path
constexpr int kStaticSplitBlocks = 1024;   // k-range parts x particle blocks of the force pass
constexpr size_t kScratchBytes = (size_t)32 << 20;
constexpr int kMaxDevices = 64;

}  // namespace

// The static path's workspaces (each GPU holds its own copy until the
// process ends).  Host code never passes this name to a kernel: it is a
// host-side stand-in, and the device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

struct StaticState {
    unsigned char *base = nullptr;   // device address of `scratch` on this device
    rbe2d_ctx h;
    rbe2d_params last{};
    bool have = false;
};
StaticState g_static[kMaxDevices];
std::mutex g_static_mu;

// Tables of one system, passed by value as kernel arguments (each launch's
// arguments stay below 4 KB)
constexpr int kFamPerPut = 32;
struct PutFam {
    Family f[kFamPerPut];
    int first, count;
};
constexpr int kImgPerPut = 32;
struct PutImg {
    double gp[kImgPerPut], gm[kImgPerPut];
    int ea_p[kImgPerPut], eb_p[kImgPerPut], ea_m[kImgPerPut], eb_m[kImgPerPut];
};
struct PutDesc {
    SysDesc d;
    int lay[10];
    PutImg img;      // the first image orders
    PutFam fam;      // the first families
};
static_assert(sizeof(PutDesc) + 128 <= 4096, "kernel arguments");

__device__ __forceinline__ void put_families(const PutFam &a, Family *fam) {
    if ((int)threadIdx.x < a.count) fam[a.first + threadIdx.x] = a.f[threadIdx.x];
}
// (the cell counts start at zero in every build: the array may hold another
// call's values)
__global__ __launch_bounds__(kBlock) void k_put_desc(PutDesc a, SysDesc *sys, int *off, int *pbase, int *bbase,
                                                     int *tbase, int *sbase, int *err, int *count, int n_count,
                                                     ImgTable *img, Family *fam) {
    for (int c = blockIdx.x * kBlock + threadIdx.x; c < n_count; c += gridDim.x * kBlock) count[c] = 0;
    if (blockIdx.x != 0) return;
    put_families(a.fam, fam);
    const int o = (int)threadIdx.x - kWave;
    if (o >= 0 && o < kImgPerPut) {
        img->gp[o] = a.img.gp[o]; img->gm[o] = a.img.gm[o];
        img->ea_p[o] = a.img.ea_p[o]; img->eb_p[o] = a.img.eb_p[o];
        img->ea_m[o] = a.img.ea_m[o]; img->eb_m[o] = a.img.eb_m[o];
    }
    if (threadIdx.x != 0) return;
    *sys = a.d;
    int *dst[5] = {off, pbase, bbase, tbase, sbase};
    for (int k = 0; k < 5; k++) {
        dst[k][0] = a.lay[2 * k];
        dst[k][1] = a.lay[2 * k + 1];
    }
    err[0] = 0;
}
__global__ void k_put_img(ImgTable a, ImgTable *img) {
    if (threadIdx.x == 0) *img = a;
}
__global__ void k_put_fam(PutFam a, Family *fam) { put_families(a, fam); }

rbe2d_status forces_noalloc(const rbe2d_params *p, const int32_t *kset, int64_t N, const double *pos,
                            const double *q, double *F, double *energy, uint32_t flags, int32_t *err_word,
                            hipStream_t s) {
    rbe2d_status st = validate(p, nullptr);
    if (st) return st;
    if (p->n_max > kStaticMaxN || p->P > kStaticMaxP)
        return fail(nullptr, RBE2D_E_INVAL,
                    "rbe2d_forces_noalloc handles n_max <= %lld and P <= %d (got n_max = %lld, P = %d)",
                    (long long)kStaticMaxN, kStaticMaxP, (long long)p->n_max, p->P);
    if (N < 0 || N > p->n_max)
        return fail(nullptr, RBE2D_E_INVAL, "N = %lld outside [0, n_max = %lld]", (long long)N,
                    (long long)p->n_max);
    if (flags & ~(uint32_t)(RBE2D_ALL | RBE2D_ACCUMULATE)) return fail(nullptr, RBE2D_E_INVAL, "unknown flags");
    if (N > 0 && (!pos || !q || !F)) return fail(nullptr, RBE2D_E_INVAL, "pos, q or F is NULL");
    if (!kset && (flags & RBE2D_KSPACE)) return fail(nullptr, RBE2D_E_INVAL, "kset is NULL");
    int dev = 0;
    const hipError_t ge = hipGetDevice(&dev);
    if (ge != hipSuccess) return hipfail(nullptr, ge, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, RBE2D_E_INVAL, "device index %d >= %d", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_static_mu);
    StaticState &S = g_static[dev];
    if (!S.base) {
        // once per device, with that device current: the array's address on it
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hipfail(nullptr, e, "hipGetSymbolAddress(scratch)");
        S.base = (unsigned char *)ptr;
    }
    rbe2d_ctx *h = &S.h;
    if (!S.have || std::memcmp(&S.last, p, sizeof *p) != 0) {
        // host set-up of the system (only when the parameters change)
        S.have = false;
        h->sys.resize(1);
        st = setup_system(p, h->sys[0]);
        if (st) return st;
        const rbe2d_params &pp = h->sys[0].p;
        SysDesc &d = h->sys[0].d;
        d.cbase = 0;
        h->n_sys = 1;
        h->batch = false;
        h->precision = pp.precision;
        h->P = pp.P;
        h->P_pad = (h->P + kPPad - 1) / kPPad * kPPad;
        h->n_cap = pp.n_max;
        h->cap_particles = std::max<int64_t>((pp.n_max + kTileMax - 1) / kTileMax * kTileMax, kTileMax);
        h->cap_sorted = std::max<int64_t>((pp.n_max + kWave - 1) / kWave * kWave, kWave);
        h->total_cells = h->max_cells = d.ncx * d.ncy * d.ncz;
        h->iso = d.iso != 0;
        h->split_blocks = kStaticSplitBlocks;
        h->one_stream = true;
        h->side = nullptr;
        // carve the workspaces from the array (no pointer of other parameters'
        // survives: FP64 has no FP32 source records, and their writer goes by
        // the pointer)
        h->w = Workspace();
        Carver carve;
        carve.base = S.base;
        plan_workspace(h, 1, false, carve);
        const size_t used = carve.used;
        if (used > kScratchBytes)
            return fail(nullptr, RBE2D_E_INVAL, "rbe2d_forces_noalloc: %zu bytes of workspace exceed the %zu-byte array",
                        used, kScratchBytes);
        S.last = *p;
        S.have = true;
    }
    h->w.kset = const_cast<int32_t *>(kset);
    h->kset_valid = true;
    int64_t cnt = N;
    PutDesc pd;
    st = compute_layout(h, &cnt, pd.lay);
    if (st) return st;
    // tables and layout: stream-ordered kernel writes (the array keeps the
    // last call's contents; every call rewrites what it reads)
    const SysHost &sh = h->sys[0];
    pd.d = sh.d;
    auto families = [&](int f0) {
        PutFam pf;
        pf.first = f0;
        pf.count = std::max(0, std::min<int>(kFamPerPut, (int)sh.fam.size() - f0));
        for (int i = 0; i < pf.count; i++) pf.f[i] = sh.fam[f0 + i];
        return pf;
    };
    pd.fam = families(0);
    for (int o = 0; o < kImgPerPut; o++) {
        pd.img.gp[o] = sh.img.gp[o]; pd.img.gm[o] = sh.img.gm[o];
        pd.img.ea_p[o] = sh.img.ea_p[o]; pd.img.eb_p[o] = sh.img.eb_p[o];
        pd.img.ea_m[o] = sh.img.ea_m[o]; pd.img.eb_m[o] = sh.img.eb_m[o];
    }
    const int ncb = std::min((h->total_cells + kBlock - 1) / kBlock, 256);
    hipLaunchKernelGGL(k_put_desc, dim3(ncb), dim3(kBlock), 0, s, pd, h->w.sys, h->w.lay.off, h->w.lay.pbase,
                       h->w.lay.bbase, h->w.lay.tbase, h->w.lay.sbase, h->w.err, h->w.count, h->total_cells, h->w.img, h->w.fam);
    if (sh.d.M > kImgPerPut) hipLaunchKernelGGL(k_put_img, dim3(1), dim3(64), 0, s, sh.img, h->w.img);
    for (int f0 = kFamPerPut; f0 < (int)sh.fam.size(); f0 += kFamPerPut)
        hipLaunchKernelGGL(k_put_fam, dim3(1), dim3(64), 0, s, families(f0), h->w.fam);
    h->cells_counted = false;
    RBE2D_TRY(nullptr, hipGetLastError(), "table upload");
    ForceJob job;
    job.energy = energy;
    job.err_out = err_word;
    st = compute_forces(h, pos, q, F, flags & RBE2D_ALL, (flags & RBE2D_ACCUMULATE) != 0, job, s);
    if (st) return fail(nullptr, st, "%s", h->err.c_str());
    RBE2D_TRY(nullptr, hipGetLastError(), "launch");
    return RBE2D_OK;
}

}  // namespace

extern "C" {

rbe2d_status rbe2d_create(const rbe2d_params *p, rbe2d_handle *out) { return create_handle(1, p, false, out); }

rbe2d_status rbe2d_batch_create(int32_t n_sys, const rbe2d_params *params, rbe2d_handle *out) {
    return create_handle(n_sys, params, true, out);
}

void rbe2d_destroy(rbe2d_handle h) {
    if (!h) return;
    int cur = 0;
    (void)hipGetDevice(&cur);
    (void)hipSetDevice(h->device);
    (void)hipDeviceSynchronize();
    free_all(h);
    (void)hipSetDevice(cur);
    delete h;
}

rbe2d_status rbe2d_query(rbe2d_handle h, double *Lz_ext, double *V, double *S) {
    return rbe2d_query_system(h, 0, Lz_ext, V, S);
}

rbe2d_status rbe2d_query_system(rbe2d_handle h, int32_t sys, double *Lz_ext, double *V, double *S) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (sys < 0 || sys >= h->n_sys) return fail(h, RBE2D_E_INVAL, "system index out of range");
    const SysDesc &d = h->sys[sys].d;
    if (Lz_ext) *Lz_ext = d.Lz;
    if (V) *V = d.V;
    if (S) *S = d.S;
    return RBE2D_OK;
}

rbe2d_status rbe2d_draw_kset(const rbe2d_params *p, uint64_t seed, uint64_t stream_id, int32_t *n_out) {
    rbe2d_status st = validate(p, nullptr);
    if (st) return st;
    if (!n_out) return fail(nullptr, RBE2D_E_INVAL, "n_out is NULL");
    const double Lz = p->Lz_ext > 0.0 ? p->Lz_ext : auto_lz(p);
    const double Ls[3] = {p->Lx, p->Ly, Lz};
    int nm[3];
    std::vector<double> cdf[3];
    for (int d = 0; d < 3; d++) axis_table(p->alpha, Ls[d], &nm[d], cdf[d]);
    const uint64_t key = stream_key(seed, stream_id);
    for (int l = 0; l < p->P; l++) {
        bool ok = false;
        for (int att = 0; att < 64 && !ok; att++) {
            const uint64_t c = ((uint64_t)l * 64 + att) * 3;
            int n[3];
            for (int d = 0; d < 3; d++) n[d] = draw_axis(cdf[d].data(), nm[d], uniform01(key, c + d));
            if (n[0] | n[1] | n[2]) {
                n_out[3 * l] = n[0]; n_out[3 * l + 1] = n[1]; n_out[3 * l + 2] = n[2];
                ok = true;
            }
        }
        if (!ok) return fail(nullptr, RBE2D_E_STATE, "k-sampler drew 64 zero vectors in a row");
    }
    return RBE2D_OK;
}

rbe2d_status rbe2d_set_kset(rbe2d_handle h, const int32_t *n, int n_is_device, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (!n) return fail(h, RBE2D_E_INVAL, "n is NULL");
    h->calls++;
    hipStream_t s = (hipStream_t)stream;
    const size_t cnt = 3 * (size_t)h->n_sys * h->P;
    if (n_is_device) {
        RBE2D_TRY(h, hipMemcpyAsync(h->w.kset, n, cnt * sizeof(int32_t), hipMemcpyDeviceToDevice, s),
                  "set_kset copy");
        h->kset_valid = true;
        return RBE2D_OK;
    }
    for (int r = 0; r < h->n_sys; r++) {
        const SysDesc &d = h->sys[r].d;
        const int64_t lim = h->precision == RBE2D_PREC_FP32_PHASE ? ((int64_t)1 << (22 - d.fh_bits))
                                                                  : ((int64_t)1 << 20);
        for (int l = 0; l < h->P; l++) {
            const int32_t *v = n + 3 * ((size_t)r * h->P + l);
            if (!(v[0] | v[1] | v[2]))
                return fail(h, RBE2D_E_INVAL, "k-set entry %d of system %d is the zero vector", l, r);
            for (int c = 0; c < 3; c++)
                if (std::llabs((long long)v[c]) >= lim)
                    return fail(h, RBE2D_E_INVAL, "k-set entry %d of system %d exceeds |n| < %lld", l, r,
                                (long long)lim);
        }
    }
    // the pinned staging buffer may still feed the previous upload
    if (h->kev_pending) RBE2D_TRY(h, hipEventSynchronize(h->kev), "set_kset wait");
    std::memcpy(h->kstage, n, cnt * sizeof(int32_t));
    RBE2D_TRY(h, hipMemcpyAsync(h->w.kset, h->kstage, cnt * sizeof(int32_t), hipMemcpyHostToDevice, s),
              "set_kset copy");
    RBE2D_TRY(h, hipEventRecord(h->kev, s), "set_kset event");
    h->kev_pending = true;
    h->kset_valid = true;
    return RBE2D_OK;
}

rbe2d_status rbe2d_sample_kset(rbe2d_handle h, uint64_t seed, uint64_t stream_id, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    h->calls++;
    RBE2D_TRY(h, launch_sample(h, seed, stream_id, nullptr, (hipStream_t)stream), "sample_kset launch");
    h->kset_valid = true;
    return RBE2D_OK;
}

rbe2d_status rbe2d_get_kset(rbe2d_handle h, int32_t *n_host, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (!n_host) return fail(h, RBE2D_E_INVAL, "n_host is NULL");
    if (!h->kset_valid) return fail(h, RBE2D_E_STATE, "no k-set");
    hipStream_t s = (hipStream_t)stream;
    RBE2D_TRY(h, hipMemcpyAsync(n_host, h->w.kset, 3 * sizeof(int32_t) * h->n_sys * h->P, hipMemcpyDeviceToHost, s),
              "get_kset copy");
    RBE2D_TRY(h, hipStreamSynchronize(s), "get_kset sync");
    return RBE2D_OK;
}

static rbe2d_status single_layout(rbe2d_ctx *h, int64_t N, hipStream_t s) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (h->batch) return fail(h, RBE2D_E_STATE, "batched handle: use the rbe2d_batch_* calls");
    return set_layout(h, &N, s);
}

rbe2d_status rbe2d_forces(rbe2d_handle h, int64_t N, const double *pos, const double *q, double *F,
                          double *energy, uint32_t flags, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = single_layout(h, N, s);
    if (st) return st;
    return run_forces(h, pos, q, F, energy, flags, s);
}

rbe2d_status rbe2d_batch_forces(rbe2d_handle h, const int64_t *offsets, const double *pos, const double *q,
                                double *F, double *energy, uint32_t flags, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = layout_from_offsets(h, offsets, s);
    if (st) return st;
    return run_forces(h, pos, q, F, energy, flags, s);
}

rbe2d_status rbe2d_energy(rbe2d_handle h, int64_t N, const double *pos, const double *q, double *energy,
                          void *stream) {
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = single_layout(h, N, s);
    if (st) return st;
    if (!energy) return fail(h, RBE2D_E_INVAL, "energy is NULL");
    const CountGuard guard{h, s};
    st = check_arrays(h, pos, q);
    if (st) return st;
    // the gamma-derivative sums of the pair kernel cost little and let a
    // following rbe2d_energy_backward reuse everything this call leaves
    st = run_common(h, pos, q, RBE2D_ALL, true, s);
    if (st) return st;
    RBE2D_TRY(h, launch_energy(h, energy, RBE2D_ALL, nullptr, nullptr, s), "energy launch");
    h->fwd.at = h->calls;
    h->fwd.pos = pos;
    h->fwd.q = q;
    h->fwd.n = N;
    return RBE2D_OK;
}

rbe2d_status rbe2d_energy_backward(rbe2d_handle h, int64_t N, const double *pos, const double *q,
                                   const double *gE, double *dEdr, double *dEdq, double *dEdgamma,
                                   void *stream) {
    hipStream_t s = (hipStream_t)stream;
    // state of an immediately preceding rbe2d_energy on the same inputs:
    // per-k records (rho, A, B), the IBC scalars and the pair kernel's
    // per-particle outputs; otherwise it is recomputed
    const bool reuse = h && h->fwd.at == h->calls && h->fwd.pos == pos && h->fwd.q == q && h->fwd.n == N;
    rbe2d_status st = single_layout(h, N, s);
    if (st) return st;
    if (!gE) return fail(h, RBE2D_E_INVAL, "gE is NULL");
    const CountGuard guard{h, s};
    st = check_arrays(h, pos, q);
    if (st) return st;
    if (!reuse) {
        st = run_common(h, pos, q, RBE2D_ALL, dEdgamma != nullptr, s);
        if (st) return st;
    }
    const bool adjoint = (dEdr || dEdq) && N > 0;
    ForceExtra x;
    x.dEdgamma = dEdgamma;
    if (adjoint)
        RBE2D_TRY(h, launch_kforce(h, pos, q, dEdr, dEdq, RBE2D_ALL, false, true, true, gE, s, x), "adjoint launch");
    else if (dEdgamma) RBE2D_TRY(h, launch_energy(h, nullptr, RBE2D_ALL, gE, dEdgamma, s), "dgamma launch");
    return RBE2D_OK;
}

rbe2d_status rbe2d_md_run(rbe2d_handle h, int64_t N, double *pos, double *vel, const double *q, double *F,
                          double dt, double z_lo, double z_hi, uint64_t seed, int64_t step0, int32_t n_steps,
                          int32_t use_graph, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = single_layout(h, N, s);
    if (st) return st;
    const SysHost &sh = h->sys[0];
    if (N > 0 && (!pos || !vel || !q || !F)) return fail(h, RBE2D_E_INVAL, "NULL array");
    if (!(dt > 0.0) || !(z_lo > 0.0 && z_lo < z_hi && z_hi < sh.p.H) || n_steps < 0)
        return fail(h, RBE2D_E_INVAL, "need dt > 0, 0 < z_lo < z_hi < H, n_steps >= 0");
    return md_run(h, pos, vel, q, F, dt, z_lo, sh.p.H - z_hi, seed, step0, n_steps, use_graph != 0, nullptr, s);
}

rbe2d_status rbe2d_batch_md_run(rbe2d_handle h, const int64_t *offsets, double *pos, double *vel, const double *q,
                                double *F, double dt, double wall_margin, uint64_t seed, int64_t step0,
                                int32_t n_steps, int32_t use_graph, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = layout_from_offsets(h, offsets, s);
    if (st) return st;
    if (h->n_total > 0 && (!pos || !vel || !q || !F)) return fail(h, RBE2D_E_INVAL, "NULL array");
    double hmin = h->sys[0].p.H;
    for (const SysHost &sh : h->sys) hmin = std::min(hmin, sh.p.H);
    if (!(dt > 0.0) || !(wall_margin > 0.0 && 2 * wall_margin < hmin) || n_steps < 0)
        return fail(h, RBE2D_E_INVAL, "need dt > 0, 0 < wall_margin < H/2, n_steps >= 0");
    return md_run(h, pos, vel, q, F, dt, wall_margin, wall_margin, seed, step0, n_steps, use_graph != 0, nullptr,
                  s);
}

rbe2d_status rbe2d_force_variance(rbe2d_handle h, const int64_t *offsets, const double *pos, const double *q,
                                  double *var, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    rbe2d_status st = layout_from_offsets(h, offsets, s);
    if (st) return st;
    st = check_arrays(h, pos, q);
    if (st) return st;
    if (h->n_total > 0 && !var) return fail(h, RBE2D_E_INVAL, "var is NULL");
    st = run_common(h, pos, q, RBE2D_KSPACE, false, s);
    if (st) return st;
    ForceExtra x;
    x.var = var;
    RBE2D_TRY(h, launch_kforce(h, pos, q, nullptr, nullptr, RBE2D_KSPACE, false, false, false, nullptr, s, x),
              "variance launch");
    return RBE2D_OK;
}

rbe2d_status rbe2d_suggest_params(int64_t N, double Lx, double Ly, double H, double gamma_top, double gamma_bot,
                                  double tol, rbe2d_params *p) {
    if (!p) return fail(nullptr, RBE2D_E_INVAL, "params is NULL");
    if (N < 1 || !finite_pos(Lx) || !finite_pos(Ly) || !finite_pos(H))
        return fail(nullptr, RBE2D_E_INVAL, "need N >= 1 and finite Lx, Ly, H > 0");
    if (!(tol > 0.0 && tol < 1.0)) return fail(nullptr, RBE2D_E_INVAL, "tol must be in (0, 1)");
    if (!(std::fabs(gamma_top) <= 1.0) || !(std::fabs(gamma_bot) <= 1.0))
        return fail(nullptr, RBE2D_E_INVAL, "|gamma_top|, |gamma_bot| must be <= 1");
    const double lg = std::log(1.0 / tol);
    // alpha ~ (N / (Lx Ly H))^(1/3), independent of Lz (Sec. 2.4)
    double alpha = std::cbrt((double)N / (Lx * Ly * H));
    // real-space tail exp(-alpha^2 r_c^2) = tol, with r_c <= min(Lx, Ly)/2
    double rc = std::sqrt(lg) / alpha;
    if (rc > 0.5 * std::min(Lx, Ly)) {
        rc = 0.5 * std::min(Lx, Ly);
        alpha = std::sqrt(lg) / rc;
    }
    // smallest M whose image truncation estimate of Theorem 3.2 is within tol
    const double decay = 2.0 * kPi * H / std::max(Lx, Ly);
    int M = 0;
    for (; M < 64; M++) {
        int a, b;
        exponents(M + 1, -1, &a, &b);   // floor((M+1)/2) of gamma_top, ceil((M+1)/2) of gamma_bot
        const double est = ipow(std::fabs(gamma_top), a) * ipow(std::fabs(gamma_bot), b) * std::exp(-decay * (M - 1));
        if (est <= tol) break;
    }
    p->alpha = alpha;
    p->r_c = rc;
    p->M = M;
    p->gamma_top = gamma_top;
    p->gamma_bot = gamma_bot;
    p->Lx = Lx; p->Ly = Ly; p->H = H;
    p->eps_lz = tol;
    p->Lz_ext = auto_lz(p);
    return RBE2D_OK;
}

rbe2d_status rbe2d_short_forces(rbe2d_handle h, const int64_t *offsets, const double *pos, const double *q,
                                double *F, double *energy, const rbe2d_md_params *mp, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    MdExtra mx;
    rbe2d_status st = md_extra(h, mp, 1.0, &mx);
    if (st) return st;
    st = layout_from_offsets(h, offsets, s);
    if (st) return st;
    if (h->n_total > 0 && (!pos || !q || !F)) return fail(h, RBE2D_E_INVAL, "NULL array");
    const CountGuard guard{h, s};
    if (mx.short_on()) RBE2D_TRY(h, launch_cells(h, pos, q, s), "cell list");
    RBE2D_TRY(h, launch_short(h, mx, F, energy, s), "short-range launch");
    return RBE2D_OK;
}

rbe2d_status rbe2d_md_run_ex(rbe2d_handle h, const int64_t *offsets, double *pos, double *vel, const double *q,
                             double *F, double dt, const rbe2d_md_params *mp, uint64_t seed, int64_t step0,
                             int32_t n_steps, int32_t use_graph, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    if (!(dt > 0.0) || n_steps < 0) return fail(h, RBE2D_E_INVAL, "need dt > 0, n_steps >= 0");
    MdExtra mx;
    rbe2d_status st = md_extra(h, mp, dt, &mx);
    if (st) return st;
    st = layout_from_offsets(h, offsets, s);
    if (st) return st;
    if (h->n_total > 0 && (!pos || !vel || !q || !F)) return fail(h, RBE2D_E_INVAL, "NULL array");
    return md_run(h, pos, vel, q, F, dt, mx.margin, mx.margin, seed, step0, n_steps, use_graph != 0, &mx, s);
}

rbe2d_status rbe2d_autotune(rbe2d_handle h, const int64_t *offsets, const double *pos, const double *q,
                            int32_t *chosen, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    if (!offsets) return fail(h, RBE2D_E_INVAL, "offsets is NULL");
    if (offsets[0] != 0) return fail(h, RBE2D_E_INVAL, "offsets[0] must be 0");
    std::vector<int64_t> counts(h->n_sys);
    for (int r = 0; r < h->n_sys; r++) {
        counts[r] = offsets[r + 1] - offsets[r];
        if (counts[r] < 0 || counts[r] > h->sys[r].p.n_max)
            return fail(h, RBE2D_E_INVAL, "system %d: N outside [0, n_max]", r);
    }
    int64_t total = 0;
    for (int64_t c : counts) total += c;
    if (!h->kset_valid) return fail(h, RBE2D_E_STATE, "no k-set: call rbe2d_set_kset or rbe2d_sample_kset");
    if (total > 0 && (!pos || !q)) return fail(h, RBE2D_E_INVAL, "pos or q is NULL");
    RBE2D_TRY(h, hipStreamSynchronize(s), "autotune sync");
    const CountGuard guard{h, s};
    free_graph(h);                 // a captured step holds the old launch parameters
    h->tune = rbe2d_ctx::Tuning();
    const int prof_n = h->prof.n;
    h->prof.n = 0;                 // the trials are not traced
    hipEvent_t e0 = nullptr, e1 = nullptr;
    rbe2d_status st = RBE2D_OK;
    hipError_t he = hipEventCreate(&e0);
    if (he == hipSuccess) he = hipEventCreate(&e1);
    // minimum over reps of the duration of the launches `fn` enqueues
    auto time = [&](auto fn, int reps, float *best) -> rbe2d_status {
        *best = 1e30f;
        for (int i = 0; i < reps; i++) {
            RBE2D_TRY(h, hipEventRecord(e0, s), "autotune event");
            RBE2D_TRY(h, fn(), "autotune launch");
            RBE2D_TRY(h, hipEventRecord(e1, s), "autotune event");
            RBE2D_TRY(h, hipEventSynchronize(e1), "autotune sync");
            float ms = 0.0f;
            RBE2D_TRY(h, hipEventElapsedTime(&ms, e0, e1), "autotune elapsed");
            *best = std::min(*best, ms);
        }
        return RBE2D_OK;
    };
    int best_per = 1, best_ks = 1, best_rs = 1;
    if (he != hipSuccess) st = hipfail(h, he, "autotune events");
    // 1. particles per thread of the structure-factor tiles
    float tbest = 1e30f;
    for (int per = kMaxTileThreads; st == RBE2D_OK && per >= 1 && total > 0; per >>= 1) {
        h->force_per = per;
        st = set_layout(h, counts.data(), s);
        float t = 0.0f;
        if (st == RBE2D_OK)
            st = time([&] {
                hipError_t e = launch_prep(h, pos, q, s);
                return e == hipSuccess ? launch_kcoef_sf(h, s) : e;
            }, 3, &t);
        if (st == RBE2D_OK && t < tbest) { tbest = t; best_per = per; }
    }
    // 2. k-range split of the force pass (the per-k records of the chosen tiling)
    h->force_per = best_per;
    if (st == RBE2D_OK) st = set_layout(h, counts.data(), s);
    if (st == RBE2D_OK && total > 0) {
        const hipError_t e = launch_prep(h, pos, q, s);
        if (e != hipSuccess) st = hipfail(h, e, "autotune prep");
        else if ((he = launch_kcoef_sf(h, s)) != hipSuccess) st = hipfail(h, he, "autotune sf");
    }
    tbest = 1e30f;
    for (int ks = 1; st == RBE2D_OK && ks <= 64 && total > 0; ks <<= 1) {
        if ((int64_t)ks * h->n_blocks > h->split_blocks) break;
        h->force_ksplit = ks;
        float t = 0.0f;
        // the real-space output array serves as scratch for the forces
        st = time([&] {
            return launch_kforce(h, pos, q, (double *)h->w.freal, nullptr, RBE2D_KSPACE, false, false, false,
                                 nullptr, s);
        }, 3, &t);
        if (st == RBE2D_OK && t < tbest) { tbest = t; best_ks = ks; }
    }
    h->force_ksplit = 0;
    // 3. split of the pair work: column groups (FP32, small systems only) or
    // waves per tile (FP64)
    tbest = 1e30f;
    for (int rs = 1; st == RBE2D_OK && rs <= (h->split_cap > 0 ? kMaxRealSplit : kTileSplits) && total > 0 &&
         (h->split_cap == 0 || total <= h->split_cap); rs++) {
        h->force_rsplit = rs;
        float t = 0.0f;
        st = time([&] { return launch_real(h, pos, q, false, s); }, 3, &t);
        if (st == RBE2D_OK && t < tbest) { tbest = t; best_rs = rs; }
    }
    h->force_rsplit = 0;
    h->force_per = 0;
    h->prof.n = prof_n;
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    if (st) return st;
    h->tune.counts = counts;
    h->tune.per = best_per;
    h->tune.ksplit = best_ks;
    h->tune.rsplit = best_rs;
    st = set_layout(h, counts.data(), s);
    if (st) return st;
    if (chosen) { chosen[0] = best_per; chosen[1] = best_ks; chosen[2] = best_rs; }
    RBE2D_TRY(h, hipStreamSynchronize(s), "autotune sync");
    return RBE2D_OK;
}

rbe2d_status rbe2d_profile_enable(rbe2d_handle h, int32_t n_events) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (n_events < 0 || n_events > (1 << 20)) return fail(h, RBE2D_E_INVAL, "n_events out of range");
    RBE2D_TRY(h, hipDeviceSynchronize(), "profile sync");
    prof_free(h);
    Profiler &p = h->prof;
    for (int sl = 0; sl < RBE2D_PROF_SLOTS; sl++)
        for (int b = 0; b < 2; b++) {
            p.ev[sl][b].resize(n_events);
            for (int i = 0; i < n_events; i++) RBE2D_TRY(h, hipEventCreate(&p.ev[sl][b][i]), "profile event");
        }
    p.n = n_events;
    p.mask = ~0u;
    return RBE2D_OK;
}

rbe2d_status rbe2d_profile_classes(rbe2d_handle h, uint32_t class_mask) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    h->prof.mask = class_mask;
    return RBE2D_OK;
}

rbe2d_status rbe2d_profile_read(rbe2d_handle h, double *ms, int64_t *launches, int32_t n_slots) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (n_slots < 0 || n_slots > RBE2D_PROF_SLOTS) return fail(h, RBE2D_E_INVAL, "n_slots out of range");
    RBE2D_TRY(h, hipDeviceSynchronize(), "profile sync");
    Profiler &p = h->prof;
    for (int sl = 0; sl < RBE2D_PROF_SLOTS; sl++) {
        double t = 0.0;
        for (int i = 0; i < p.used[sl]; i++) {
            float f = 0.0f;
            RBE2D_TRY(h, hipEventElapsedTime(&f, p.ev[sl][0][i], p.ev[sl][1][i]), "profile elapsed");
            t += f;
        }
        if (sl < n_slots) {
            if (ms) ms[sl] = t;
            if (launches) launches[sl] = p.used[sl];
        }
        p.used[sl] = 0;
    }
    return RBE2D_OK;
}

rbe2d_status rbe2d_forces_noalloc(const rbe2d_params *p, const int32_t *kset, int64_t N, const double *pos,
                                  const double *q, double *F, double *energy, uint32_t flags, int32_t *err_word,
                                  void *stream) {
    return forces_noalloc(p, kset, N, pos, q, F, energy, flags, err_word, (hipStream_t)stream);
}

rbe2d_status rbe2d_set_surface_charges(rbe2d_handle h, int32_t sys, double sigma_top, double sigma_bot) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    if (sys < -1 || sys >= h->n_sys) return fail(h, RBE2D_E_INVAL, "system index out of range");
    if (!std::isfinite(sigma_top) || !std::isfinite(sigma_bot))
        return fail(h, RBE2D_E_INVAL, "surface charge densities must be finite");
    for (int r = 0; r < h->n_sys; r++) {
        if (sys >= 0 && r != sys) continue;
        h->sys[r].d.sig_top = sigma_top;
        h->sys[r].d.sig_bot = sigma_bot;
        surface_setup(h->sys[r]);
    }
    h->calls++;
    std::vector<SysDesc> descs(h->n_sys);
    for (int r = 0; r < h->n_sys; r++) descs[r] = h->sys[r].d;
    RBE2D_TRY(h, hipDeviceSynchronize(), "surface charges sync");
    RBE2D_TRY(h, hipMemcpy(h->w.sys, descs.data(), h->n_sys * sizeof(SysDesc), hipMemcpyHostToDevice),
              "surface charges upload");
    return RBE2D_OK;
}

rbe2d_status rbe2d_check(rbe2d_handle h, void *stream) {
    if (!h) return fail(nullptr, RBE2D_E_INVAL, "handle is NULL");
    hipStream_t s = (hipStream_t)stream;
    RBE2D_TRY(h, hipStreamSynchronize(s), "check sync");
    RBE2D_TRY(h, hipGetLastError(), "asynchronous kernel error");
    int word = 0;
    RBE2D_TRY(h, hipMemcpy(&word, h->w.err, sizeof(int), hipMemcpyDeviceToHost), "check read");
    if (word) RBE2D_TRY(h, hipMemset(h->w.err, 0, sizeof(int)), "check clear");
    if (word & 1) return fail(h, RBE2D_E_RANGE, "a particle had z outside (0, H)");
    if (word & 2) return fail(h, RBE2D_E_STATE, "device k-sampler drew 64 zero vectors in a row");
    return RBE2D_OK;
}

const char *rbe2d_last_error(rbe2d_handle h) {
    if (!h) return g_create_error.c_str();
    return h->err.c_str();
}

}  // extern "C"
