// Pair sums over tiles of targets on gfx950: the FP64 erfc sum of real charges
// and images (Eq. (3.12)) and the short-range repulsion of the MD, both in
// FP64 on the cell list of realspace.hip.
#include <algorithm>

#include "devmath.h"
#include "erfcx_fit.h"
#include "exp2_fit.h"
#include "kspace_dev.h"
#include "rbe2d_internal.h"

namespace rbe2d {

// ---------------------------------------------------------------------------
// Pair sums.  A tile is 64 consecutive targets of one system in cell order
// (one lane each); 1 to 64 waves share its candidates.
//
//  1. The columns of cells that come within the cutoff of the tile's bounding
//     box -- in the periodic copies and, for the erfc sum, in every image
//     family -- give runs of consecutive sorted sources (RunFinder, one
//     column per lane).
//  2. The runs together are one list of candidates.  A chunk takes 64 of them,
//     one per lane and evenly spread over the list, so that every target finds
//     about the same share of its neighbours in each chunk: a lane that is
//     ahead waits for little.  (In list order a chunk is one column, near some
//     targets and out of reach of the others: 0.53 of the lanes busy in the
//     pair rounds instead of 0.87, with two chunks in flight.)
//  3. One MFMA per 32 x 32 block gives |s|^2 - 2 s.t + |t|^2 - R^2 for all
//     64 x 64 candidate pairs, in half precision about the tile's centre with
//     R widened by the rounding: no pair in reach is missed, and the 1 to 2 %
//     too many are dropped by the exact FP64 test of step 4.  The sign bits
//     become one 64-bit word per target: one v_alignbit per candidate, where
//     an FP64 displacement test is about ten instructions.
//  4. Rounds: every lane takes the lowest bit of its word, reads that source
//     from LDS, forms the FP64 displacement and adds its terms.  Lanes that
//     finish a chunk go on with the next one; a chunk is staged when no lane
//     needs the oldest of the two any more.
//
// Image sources are staged at their image positions with their weights
// applied to the charge, so real charges and images share the rounds.
//
// Bound by VALU issue (0.81 of the issue slots at 3 waves per SIMD; at 4 the
// pair terms spill).  1e6-ion slab, 164 pairs per target out of 1390
// candidates: 0.77 ms, where one scan of cells per target with FP64 tests and
// a wave-wide queue took 1.40 ms; 1e4 ions between two dielectric jumps 54
// instead of 171 us, 500 ions 25 instead of 44 us.
// ---------------------------------------------------------------------------

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16 __attribute__((ext_vector_type(16)));

enum TileKind { kErfc, kWca };

struct TileArgs {
    const double4 *src;         // sorted sources: (x wrapped, y wrapped, z, q)
    const int *sidx, *start;
    const SysDesc *sys;
    const Family *fam;          // kMaxFamilies per system
    Layout lay;
    int n_sys, n_total, n_waves;   // n_waves: tiles of all systems
    int wpt;                    // waves per tile in a block
    int parts;                  // blocks (grid rows) per tile; their sums go to freal_s and rpart_s if > 1
    double4 *freal_s;
    double *rpart_s;
    int nblocks;                // logical blocks (the grid is rounded up to 8 * kTileChunks chunks)
    int nbx;                    // ASM: blocks that sum pairs
    double4 *freal;
    double *rpart;              // per tile
    // short-range forces
    MdExtra mx;
    double *F;                  // added to when set, else written to freal
    double *spart;              // per tile
};

constexpr int kTileChunks = 8;      // contiguous tile ranges per XCD
constexpr int kMaxRuns = 80;        // runs per batch of the candidate list
constexpr int kRunGroup = 16;       // columns looked up together; up to 3 runs each
constexpr int kMaxTileWaves = 12;   // waves per tile (and block)

// LDS written by other lanes of the same wave: the wave's LDS operations are
// executed in order, this keeps the compiler from reordering them
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Constants of the FP64 pair terms.
struct PairConst64 {
    double a, c2a;      // alpha, 2 alpha / sqrt(pi)
    double ch, cl;      // -alpha^2 log2(e) in two parts
    bool clip;          // alpha r_c beyond the fitted range of erfcx
    __device__ PairConst64(double alpha, double rc) : a(alpha), c2a(1.1283791670955126 * alpha) {
        constexpr double l2h = 1.4426950408889634, l2l = 2.0355273740931033e-17;   // log2(e)
        const double a2h = alpha * alpha, a2l = fma(alpha, alpha, -a2h);
        const double h = a2h * l2h;
        ch = uniform(-h);
        cl = uniform(-(fma(a2h, l2h, -h) + fma(a2h, l2l, a2l * l2h)));
        clip = alpha * rc >= RBE2D_ERFCX_XMAX;
    }
};
// FP64: erfc(x) = exp(-x^2) erfcx(x) with the fitted erfcx (relative error
// below 2e-11), sharing the exponential of the force term; for x beyond the
// fitted range erfc(x) < 1.2e-29 and the term is dropped.  1/sqrt(r^2) and
// 1/(1 + p x) are the hardware estimates (2^-24) with one third-order step
// each (relative error near 1e-16; r^2 > 0 for every accepted pair); the
// exponential is 2^(-alpha^2 log2(e) r^2) with the exponent's rounding error
// carried along and the polynomial of exp2_fit.h.
// The coefficients are read from LDS (`coef`, a copy of rbe2d_erfcx64_a): as
// FP64 literals they would hold 24 registers for the whole kernel.
__device__ __forceinline__ void pair_terms(double r2, const PairConst64 &c, double *ec, double *fs,
                                           const double *coef) {
    double y = __builtin_amdgcn_rsq(r2);
    const double en = fma(-r2 * y, y, 1.0);     // 1 - r^2 y^2
    y = fma(y * en, fma(0.375, en, 0.5), y);
    const double d = r2 * y;
    const double rinv2 = y * y;
    const double n = rint(c.ch * r2);
    const double f = fma(c.cl, r2, fma(c.ch, r2, -n));
    double e = kExp2[kExp2Terms - 1];
#pragma unroll
    for (int k = kExp2Terms - 2; k >= 0; k--) e = fma(e, f, kExp2[k]);
    e = __builtin_amdgcn_ldexp(fma(f, e, 1.0), (int)n);
    const double x = c.a * d;
    const double a1 = fma(RBE2D_ERFCX64_P, x, 1.0);
    double t = __builtin_amdgcn_rcp(a1);
    const double et = fma(-a1, t, 1.0);
    t = fma(t, fma(et, et, et), t);
    double p = coef[RBE2D_ERFCX64_DEG - 1];
#pragma unroll
    for (int k = RBE2D_ERFCX64_DEG - 2; k >= 0; k--) p = fma(p, t, coef[k]);
    double v = e * (p * t) * y;
    if (c.clip) v = x < RBE2D_ERFCX_XMAX ? v : 0.0;
    *ec = v;
    *fs = fma(c.c2a, e, v) * rinv2;
}

__device__ __forceinline__ double lj_rep(double s2_over_r2, double eps, double *r_times_f) {
    const double s6 = s2_over_r2 * s2_over_r2 * s2_over_r2;
    *r_times_f = 24.0 * eps * (2.0 * s6 * s6 - s6);
    return 4.0 * eps * (s6 * s6 - s6 + 0.25);
}

// Energy of an ion at height z at the two walls, its force added to fz
__device__ __forceinline__ double wall_terms(const MdExtra &mx, const SysDesc &d, double z, double *fz) {
    double ew = 0.0, rf;
    if (mx.epsw != 0.0) {
        const double hb = z, ht = d.H - z;
        if (hb > 0.0 && hb < mx.hcut) { ew += lj_rep(mx.sigw2 / (hb * hb), mx.epsw, &rf); *fz += rf / hb; }
        if (ht > 0.0 && ht < mx.hcut) { ew += lj_rep(mx.sigw2 / (ht * ht), mx.epsw, &rf); *fz -= rf / ht; }
    }
    return ew;
}

// of nonnegative floats, whose bits order like integers
__device__ __forceinline__ float wave_fmin(float v, bool on) {
    return __int_as_float(wave_reduce<false>(on ? __float_as_int(v) : 0x7f800000));
}
__device__ __forceinline__ float wave_fmax(float v, bool on) {
    return __int_as_float(wave_reduce<true>(on ? __float_as_int(v) : 0));
}

// One image family as a placement of sources: z' = s z + c with weight w
// (f = 0: the real charges).  The tables hold it from the target's side.
struct Placement {
    double c, w, wt, wb;
    bool mirror;   // s = -1
};
__device__ __forceinline__ Placement placement(const Family *fams, int f) {
    Placement p{0.0, 1.0, 0.0, 0.0, false};
    if (f > 0) {
        const Family fm = fams[f - 1];
        p.mirror = fm.sz < 0.0;
        p.c = p.mirror ? fm.cz : -fm.cz;
        p.w = fm.w; p.wt = fm.dwt; p.wb = fm.dwb;
    }
    return p;
}

// A run of candidates and the placement of its sources (LDS).
struct Run {
    int off, end;              // list position - off = sorted index; last position + 1
    int code;                  // image family | (x copy + 1) << 8 | (y copy + 1) << 10
    int pad;
    float shx, shy, zm, za;    // prefilter coordinates: x + shx, y + shy, zm z + za
    double c, w;               // placement: height shift and weight; the mirror is the sign of zm
};
constexpr int kSelfCode = 0 | 1 << 8 | 1 << 10;   // real charges, no shift
__device__ __forceinline__ int copy_x(int code) { return ((code >> 8) & 3) - 1; }
__device__ __forceinline__ int copy_y(int code) { return ((code >> 10) & 3) - 1; }

// The runs of a tile: for every image family and every column of cells within
// the cutoff of the tile's bounding box, the cells along y that the cutoff
// leaves, as consecutive sorted positions.  Columns and cells are counted
// without wrapping: copies by one period (the box lies in the cell, and the
// cutoff is at most half a period) carry their shift in the run's code.
// Bounds are in FP32, widened by `marg` against their rounding: they only
// decide which cells are candidates.
template <bool DG>
struct RunFinder {
    const SysDesc &d;
    const Family *fams;
    const int *start;
    Run *runs;                      // LDS; entry kMaxRuns: the tile's own targets
    double2 *dgw;                   // LDS (DG): gamma derivatives of the runs' weights
    float x0, x1, y0, y1, z0, z1;   // bounding box of the tile
    float rcm, marg;
    float xc, yc, zc;               // centre of the prefilter's frame
    int nfam, shift, lane, cxlo, ncol;
    int f = 0, i0 = 0;              // next family and column group
    int nr = 0, total = 0;          // runs and candidates of the current batch

    __device__ __forceinline__ void put(int k, int o, int e, int code, const Placement &p) {
        Run r;
        r.off = o; r.end = e; r.code = code;
        r.shx = (float)copy_x(code) * (float)d.Lx - xc;
        r.shy = (float)copy_y(code) * (float)d.Ly - yc;
        r.zm = p.mirror ? -1.0f : 1.0f;
        r.za = (float)p.c - zc;
        r.pad = 0;
        r.c = p.c; r.w = p.w;
        runs[k] = r;
        if (DG) dgw[k] = make_double2(p.wt, p.wb);
    }

    // the next batch of runs; false when none is left
    __device__ __forceinline__ bool fill() {
        nr = total = 0;
        while (f <= nfam && nr <= kMaxRuns - 3 * kRunGroup) {
            const Placement p = placement(fams, f);
            const float c = (float)p.c, hz = (float)d.hz, inv_hz = (float)d.inv_hz;
            // heights of real sources whose images come within the cutoff
            const float za = p.mirror ? c - z1 - rcm : z0 - rcm - c;
            const float zb = p.mirror ? c - z0 + rcm : z1 + rcm - c;
            const int l0 = max(0, (int)floorf(fmaxf(za * inv_hz, -1.0f)));
            const int l1 = min(d.ncz - 1, (int)floorf(fminf(zb * inv_hz, (float)d.ncz)));
            const int items = max(0, l1 - l0 + 1) * ncol;
            if (i0 >= items) { f++; i0 = 0; continue; }
            const int it = i0 + lane;
            bool on = lane < kRunGroup && it < items;
            const int li = on ? it / ncol : 0;
            const int lz = l0 + li, cx = cxlo + (it - li * ncol);
            const int sx = cx < 0 ? -1 : (cx >= d.ncx ? 1 : 0);
            const int cxw = cx - sx * d.ncx;
            const float ca = (float)cx * (float)d.hx, cb = ca + (float)d.hx;
            const float la = p.mirror ? c - (float)(lz + 1) * hz : (float)lz * hz + c, lb = la + hz;
            const float dx = fmaxf(0.0f, fmaxf(ca - x1, x0 - cb) - marg);
            const float dz = fmaxf(0.0f, fmaxf(la - z1, z0 - lb) - marg);
            const float ye2 = rcm * rcm - dx * dx - dz * dz;
            on = on && ye2 > 0.0f;
            const float ye = __builtin_amdgcn_sqrtf(fmaxf(ye2, 0.0f)) + marg;
            const float inv_hy = (float)d.inv_hy;
            const int cylo = (int)floorf((y0 - ye) * inv_hy), cyhi = (int)floorf((y1 + ye) * inv_hy);
            const int col = column_of(d, cxw, lz);
            for (int sy = -1; sy <= 1; sy++) {
                const int lo = max(cylo - sy * d.ncy, 0), hi = min(cyhi - sy * d.ncy, d.ncy - 1);
                const bool v = on && lo <= hi;
                if (__ballot(v) == 0) continue;
                int jb = 0, len = 0;
                if (v) {
                    const int c0 = cells_from(d, col, lo, hi);
                    jb = start[c0];
                    len = start[c0 + hi - lo + 1] - jb;
                }
                int incl = len;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int u = __shfl_up(incl, o, 64);
                    if (lane >= o) incl += u;
                }
                const uint64_t m = __ballot(len > 0);
                if (len > 0) {
                    const int k = nr + __popcll(m & ((1ull << lane) - 1ull));
                    put(k, total + incl - len - (jb + shift), total + incl, f | (sx + 1) << 8 | (sy + 1) << 10, p);
                }
                nr += __popcll(m);
                total += __builtin_amdgcn_readlane(incl, 63);
            }
            i0 += kRunGroup;
        }
        wave_lds_fence();
        return nr > 0;
    }
};

// count of trailing zeros, all ones for 0
__device__ __forceinline__ uint32_t ctz32(uint32_t v) {
    uint32_t n;
    asm("v_ffbl_b32 %0, %1" : "=v"(n) : "v"(v));
    return n;
}

// LDS of one wave: the staged sources of two chunks, with DG also their
// charges times the gamma derivatives of the weights; the targets' half-
// precision coordinates; the runs
template <bool DG>
struct TileLds {
    static constexpr int kDg = 2 * kWave * (int)sizeof(double4);
    static constexpr int kTargets = kDg + (DG ? 2 * kWave * (int)sizeof(double2) : 0);
    static constexpr int kRuns = kTargets + (kWave + 1) * (int)sizeof(half8);
    static constexpr int kDgw = kRuns + (kMaxRuns + 1) * (int)sizeof(Run);
    static constexpr int kUsed = kDgw + (DG ? (kMaxRuns + 1) * (int)sizeof(double2) : 0);
    static constexpr int kSums = 6 * kWave * (int)sizeof(double);   // aliases the rest after the last round
    static constexpr int kWaveBytes = ((kUsed > kSums ? kUsed : kSums) + 31) / 32 * 32;
};

// DG: also the gamma derivatives of the potential.
// ASM: the per-k assembly of the call rides along (blocks from nbx on), which on
// one stream waits for the pair sums otherwise.
template <TileKind KIND, bool DG, bool ASM>
__global__ __launch_bounds__(kWave * kMaxTileWaves) __attribute__((amdgpu_waves_per_eu(3, 8)))
void k_tile(TileArgs a, AssembleArgs as) {
    using Lds = TileLds<DG>;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double coef64[KIND == kErfc ? RBE2D_ERFCX64_DEG : 1];
    const int nbx = ASM ? a.nbx : (int)gridDim.x;
    if constexpr (ASM) {
        if ((int)blockIdx.x >= nbx) {
            const int b = ((int)blockIdx.x - nbx) * gridDim.y + blockIdx.y;
            assemble_wave<DG>(as, b * (blockDim.x / kWave) +
                                      __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), threadIdx.x % kWave);
            return;
        }
    }
    if (KIND == kErfc) {
        if (threadIdx.x < RBE2D_ERFCX64_DEG) coef64[threadIdx.x] = rbe2d_erfcx64_a[threadIdx.x];
        __syncthreads();
    }
    const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    // Blocks are dealt round-robin to the 8 XCDs.  Each XCD runs C contiguous
    // ranges of tiles (range k of XCD x is range 8k + x), so neighbouring
    // cells share that XCD's L2, and the tiles near the walls (cell order is
    // z-slowest; they have image sources too) are shared by all XCDs.
    const int cs = (nbx >> 3) / kTileChunks;   // blocks per range
    const int jblk = (int)(blockIdx.x >> 3);
    const int lb = ((jblk / cs) * 8 + (int)(blockIdx.x & 7)) * cs + jblk % cs;
    if (lb >= a.nblocks) return;
    const int per_block = (int)(blockDim.x / kWave) / a.wpt;
    const int tile = lb * per_block + wid / a.wpt, bsub = wid % a.wpt;
    const int sub = (int)blockIdx.y * a.wpt + bsub, nsub = (int)gridDim.y * a.wpt;   // of the tile's waves
    const bool tile_on = tile < a.n_waves;                 // wave-uniform; barriers below see every wave
    const int t = min(tile, a.n_waves - 1) * kWave + lane;
    const int r = __builtin_amdgcn_readfirstlane(find_sys(a.lay.sbase, a.n_sys, t & ~(kWave - 1)));
    const SysDesc d = a.sys[r];   // a copy: loop-invariant values stay in registers
    const Family *fams = a.fam + (int64_t)r * kMaxFamilies;
    const bool active = tile_on && t - a.lay.sbase[r] < a.lay.off[r + 1] - a.lay.off[r];
    double4 me = make_double4(0.0, 0.0, 0.0, 0.0);
    if (active) me = a.src[t];
    // an ion whose position is not finite (x and y, once wrapped, are then NaN)
    // has no pairs, and no part in the tile's box
    const bool placed = active && me.x == me.x && me.y == me.y;
    double fx = 0, fy = 0, fz = 0, phi = 0, dpt = 0, dpb = 0;
    unsigned char *wl = lds + wid * Lds::kWaveBytes;
    // all pairs of the targets `on` (the sources are the same for any of them)
    auto pass = [&](bool on) {
        double4 *ring = reinterpret_cast<double4 *>(wl);
        double2 *ringdg = reinterpret_cast<double2 *>(wl + Lds::kDg);
        half8 *tgt = reinterpret_cast<half8 *>(wl + Lds::kTargets);   // entry kWave: zeros
        Run *runs = reinterpret_cast<Run *>(wl + Lds::kRuns);
        double2 *dgw = reinterpret_cast<double2 *>(wl + Lds::kDgw);
        const float rc = KIND == kWca ? (float)sqrt(a.mx.rc2) : (float)d.rc;
        const float Lx = (float)d.Lx, Ly = (float)d.Ly;
        const float marg = 1e-5f * rc + 1e-6f * (fmaxf(Lx, Ly) + 4.0f * (float)d.H + rc);
        const float zb = fminf(fmaxf((float)me.z, 0.0f), (float)d.H);
        const float x0 = wave_fmin((float)me.x, on), x1 = wave_fmax((float)me.x, on);
        const float y0 = wave_fmin((float)me.y, on), y1 = wave_fmax((float)me.y, on);
        const float z0 = wave_fmin(zb, on), z1 = wave_fmax(zb, on);
        const float xc = 0.5f * (x0 + x1), yc = 0.5f * (y0 + y1), zc = 0.5f * (z0 + z1);
        RunFinder<DG> rf{d, fams, a.start + d.cbase, runs, dgw, x0, x1, y0, y1, z0, z1, rc + marg, marg,
                           xc, yc, zc, KIND == kWca ? 0 : d.nfam, a.lay.sbase[r] - a.lay.off[r], lane, 0, 0};
        // (columns of the box and its copies only: in a box 5e5 times as long as
        // it is wide the margin alone reaches past them)
        rf.cxlo = max((int)floorf((rf.x0 - rf.rcm) * (float)d.inv_hx), -d.ncx);
        rf.ncol = min((int)floorf((rf.x1 + rf.rcm) * (float)d.inv_hx), 2 * d.ncx - 1) - rf.cxlo + 1;
        // Prefilter frame: coordinates about the box centre, scaled by a power
        // of two so that every candidate lies within 64 (|s|^2 < 12288 in half
        // precision).  Half-precision rounding moves each coordinate by at
        // most 2^-6 there, a distance by 4 sqrt(3)/2 2^-6 = 0.055, and the two
        // split squares by 0.01; coordinates from FP32 lose up to 2^-23 of the
        // box more.  The cutoff is widened by that.
        const float ext = 0.5f * fmaxf(fmaxf(x1 - x0, y1 - y0), z1 - z0) + rf.rcm + 2.0f * marg +
                          fmaxf(fmaxf((float)d.hx, (float)d.hy), (float)d.hz);
        const float sg = __builtin_amdgcn_ldexpf(1.0f, 5 - __builtin_amdgcn_frexp_expf(ext) + 1);
        const float rs = rc * sg + 0.06f + sg * 4e-7f * (fmaxf(Lx, Ly) + 4.0f * (float)d.H + 4.0f * rc);
        const float thr = rs * rs + 0.03f;
        {
            const _Float16 hx = (_Float16)(((float)me.x - xc) * sg), hy = (_Float16)(((float)me.y - yc) * sg),
                           hz = (_Float16)(((float)me.z - zc) * sg);
            const float T = (float)hx * (float)hx + (float)hy * (float)hy + (float)hz * (float)hz - thr;
            const _Float16 th = (_Float16)T, tl = (_Float16)(T - (float)th), one = (_Float16)1.0f, two = (_Float16)-2.0f;
            half8 tv = {two * hx, two * hy, two * hz, one, one, th, tl, (_Float16)0.0f};
            if (!on) tv = half8{0, 0, 0, one, one, (_Float16)30000.0f, 0, 0};
            tgt[lane] = tv;
            if (lane == 0) {
                tgt[kWave] = half8{0, 0, 0, 0, 0, 0, 0, 0};
                rf.put(kMaxRuns, 0, 0, kSelfCode, Placement{0.0, 1.0, 0.0, 0.0, false});
            }
            wave_lds_fence();
        }
        // Operands of the four MFMAs of a chunk: lanes 0-31 hold the first 8
        // of the 16 products, lanes 32-63 the others.  Sources 0-31 sit in the
        // lower lanes and meet the targets there and zeros above, sources
        // 32-63 the other way round.
        const half8 *tlo = tgt + (lane < 32 ? lane : kWave), *thi = tgt + (lane < 32 ? kWave : lane - 32);
        const int tlo2 = lane < 32 ? 32 : 0, thi2 = lane < 32 ? 0 : 32;
        // the slot of this lane's source in its chunk, so that slot k is bit k
        // of the target's word (from the rows an MFMA leaves in each lane)
        const int srow = lane & 31;
        const int slot = ((srow >> 2) & 1) * 32 + 31 - ((lane >> 5) * 16 + (srow >> 3) * 4 + (srow & 3));
        const int t0 = t - lane;

        const PairConst64 pc64(d.alpha, d.rc);
        const double rc2 = KIND == kWca ? a.mx.rc2 : d.rc2;
        uint32_t ca = 0, cb = 0, na = 0, nb = 0;   // words of the oldest and the newest chunk
        constexpr uint32_t kRec = sizeof(double4);
        uint32_t cbase = 0;                         // byte offset of the slots of the word in ca, cb

        // one round: the lowest bit of the lane's word
        auto round = [&]() {
            const uint32_t e = min(ctz32(ca), ctz32(cb) + 32u);
            const unsigned char *rec = wl + (e * kRec + cbase);
            const uint64_t m = ((uint64_t)cb << 32 | ca), m1 = m & (m - 1ull);
            ca = (uint32_t)m1; cb = (uint32_t)(m1 >> 32);
            const double4 s = *reinterpret_cast<const double4 *>(rec);
            const double dx = me.x - s.x, dy = me.y - s.y, dz = me.z - s.z;
            const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
            if (r2 < rc2) {
                if constexpr (KIND == kErfc) {
                    double ec, fs;
                    pair_terms(r2, pc64, &ec, &fs, coef64);
                    const double qf = s.w * fs;
                    fx = fma(qf, dx, fx); fy = fma(qf, dy, fy); fz = fma(qf, dz, fz); phi = fma(s.w, ec, phi);
                    if (DG) {
                        const double2 g = ringdg[e + cbase / kRec];
                        dpt = fma(g.x, ec, dpt); dpb = fma(g.y, ec, dpb);
                    }
                } else {
                    double rfo;
                    const double ri = 1.0 / r2;
                    phi += 0.5 * lj_rep(a.mx.sig2 * ri, a.mx.eps, &rfo);
                    rfo *= ri;
                    fx = fma(rfo, dx, fx); fy = fma(rfo, dy, fy); fz = fma(rfo, dz, fz);
                }
            }
        };
        // this lane's cursor in the candidate list
        int roff = 0, rend = 0, ri = kMaxRuns;
        int src_j = t0;
        bool src_ok = false;
        double4 rec;
        // Fetches this lane's source of the next chunk; false after the last.
        // The first chunk of the tile (wave 0) is its own targets; then lane l
        // takes positions l nch + c of the list of nch chunks; the chunks of all
        // lists are dealt to the tile's waves in turn
        bool own = sub == 0, diag = false;
        int c = own ? -1 : sub - 1 - nsub, nch = 0;
        auto fetch = [&]() -> bool {
            diag = own;
            if (own) {
                own = false;
                src_ok = active;
                src_j = active ? t : t0;
            } else {
                c += nsub;
                if (c >= nch) {
                    do {
                        c -= nch;
                        if (!rf.fill()) return false;
                        nch = (rf.total + kWave - 1) / kWave;
                    } while (c >= nch);
                    int lo = 0, hi = rf.nr - 1;   // first run that ends after the lane's first position
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (runs[mid].end > lane * nch + c) hi = mid; else lo = mid + 1;
                    }
                    ri = lo - 1;
                    rend = 0;
                }
                const int p = lane * nch + c;
                const bool in = p < rf.total;
                while (in && p >= rend) {
                    ri++;
                    roff = runs[ri].off; rend = runs[ri].end;
                }
                src_j = in ? p - roff : t0;
                src_ok = in;
                if (!in) ri = kMaxRuns;   // a placement inside the box
            }
            rec = a.src[src_j];
            return true;
        };
        // stages the fetched sources and tests them against the targets
        auto stage = [&](uint32_t base) {
            const uint32_t e = base + slot;
            const Run rn = runs[ri];
            // (the tile's own targets are taken by the first chunk)
            if (!diag && rn.code == kSelfCode && (uint32_t)(src_j - t0) < (uint32_t)kWave) src_ok = false;
            const bool mirror = rn.zm < 0.0f;
            float px = (float)rec.x + rn.shx, py = (float)rec.y + rn.shy, pz = fmaf((float)rec.z, rn.zm, rn.za);
            const double xs = (double)copy_x(rn.code) * d.Lx, ys = (double)copy_y(rn.code) * d.Ly;
            ring[e] = make_double4(rec.x + xs, rec.y + ys, (mirror ? -rec.z : rec.z) + rn.c, rn.w * rec.w);
            if (DG) ringdg[e] = make_double2(dgw[ri].x * rec.w, dgw[ri].y * rec.w);
            px *= sg; py *= sg; pz *= sg;
            // kept finite (two sources share a row of the MFMAs), and as far out of
            // reach: sources without a place, and the tile's own members of another
            // pass, which may lie anywhere
            px = __builtin_amdgcn_fmed3f(px, -100.0f, 100.0f);
            py = __builtin_amdgcn_fmed3f(py, -100.0f, 100.0f);
            pz = __builtin_amdgcn_fmed3f(pz, -100.0f, 100.0f);
            const _Float16 hx = (_Float16)px, hy = (_Float16)py, hz = (_Float16)pz;
            const float S = (float)hx * (float)hx + (float)hy * (float)hy + (float)hz * (float)hz;
            const _Float16 sh = (_Float16)(src_ok ? S : 30000.0f), one = (_Float16)1.0f;
            const _Float16 sl = (_Float16)(src_ok ? S - (float)sh : 0.0f);
            const half8 av = {hx, hy, hz, sh, sl, one, one, (_Float16)0.0f};
            const float16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            uint32_t w[2] = {0, 0};
#pragma unroll
            for (int h = 0; h < 2; h++) {   // targets 0-31, 32-63 against sources 0-31 (d0), 32-63 (d1)
                const float16 d0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, tlo[h * tlo2], zero, 0, 0, 0);
                const float16 d1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, thi[h * thi2], zero, 0, 0, 0);
#pragma unroll
                for (int k = 0; k < 16; k++)
                    w[h] = __builtin_amdgcn_alignbit(w[h], __float_as_uint(d0[k]), 31);
#pragma unroll
                for (int k = 0; k < 16; k++)
                    w[h] = __builtin_amdgcn_alignbit(w[h], __float_as_uint(d1[k]), 31);
                __builtin_amdgcn_sched_barrier(0);   // two blocks' accumulators at a time
            }
            // lane l < 32 holds half of the rows of targets l and l + 32, lane
            // l + 32 the other half: exchange, so that a lane has its target's
            auto sw = __builtin_amdgcn_permlane32_swap(w[0], w[1], false, false);
            na = sw[0]; nb = sw[1];
            if (diag) {   // a target is not its own source
                if (slot < 32) na &= ~(1u << slot);
                else nb &= ~(1u << (slot - 32));
            }
            wave_lds_fence();
        };
        uint32_t nbase = 0;                        // first slot of the newest chunk
        bool more = fetch();
        for (;;) {
            const bool last = !more;   // nothing left to stage: the rounds empty the words
            na = nb = 0;
            if (more) {
                stage(nbase);
                more = fetch();
            }
            // rounds until every lane has left the oldest chunk; lanes that
            // leave it go on with the newest one
            uint64_t old = __ballot(true);
            for (;;) {
                uint64_t live = __ballot((ca | cb) != 0);
                const uint64_t sw = old & ~live;
                if (sw != 0) {
                    if (__builtin_amdgcn_inverse_ballot_w64(sw)) { ca = na; cb = nb; cbase = nbase * kRec; }
                    old &= ~sw;
                    if (old == 0) break;
                    live = __ballot((ca | cb) != 0);
                }
                if (__builtin_amdgcn_inverse_ballot_w64(live)) round();
            }
            if (last) break;
            nbase ^= kWave;
        }
    };
    if constexpr (KIND == kErfc) {
        if (__ballot(placed) != 0) pass(placed);
    } else if (a.mx.eps != 0.0) {
        // without the serpentine numbering a tile that runs over the end of a
        // layer spans all of it: one pass per layer then (21,000 ions in a thin
        // slab: 18 us instead of 102)
        const int layer = d.snake ? 0 : min(d.ncz - 1, max(0, (int)(me.z / d.hz)));
        for (uint64_t left = __ballot(placed); left != 0;) {
            const int l0 = __builtin_amdgcn_readlane(layer, (int)__builtin_ctzll(left));
            const bool on = placed && layer == l0;
            left &= ~__ballot(on);
            pass(on);
            wave_lds_fence();
        }
    }
    if (a.wpt > 1) {
        // sums of the block's waves, in wave order
        __syncthreads();
        double *mine = reinterpret_cast<double *>(wl);
        if (bsub != 0) {
            mine[lane] = fx; mine[kWave + lane] = fy; mine[2 * kWave + lane] = fz; mine[3 * kWave + lane] = phi;
            if (DG) { mine[4 * kWave + lane] = dpt; mine[5 * kWave + lane] = dpb; }
        }
        __syncthreads();
        if (bsub != 0) return;
        for (int s = 1; s < a.wpt; s++) {
            const double *o = reinterpret_cast<const double *>(wl + s * Lds::kWaveBytes);
            fx += o[lane]; fy += o[kWave + lane]; fz += o[2 * kWave + lane]; phi += o[3 * kWave + lane];
            if (DG) { dpt += o[4 * kWave + lane]; dpb += o[5 * kWave + lane]; }
        }
    }
    if (!tile_on) return;
    if constexpr (KIND == kWca) {
        double ep = phi, ew = 0.0;
        if (active) {
            ew = wall_terms(a.mx, d, me.z, &fz);
            if (a.F) {
                double *o = a.F + (int64_t)3 * a.sidx[t];
                o[0] += fx; o[1] += fy; o[2] += fz;
            } else {
                a.freal[a.sidx[t]] = make_double4(fx, fy, fz, 0.0);
            }
        }
        ep = wave_sum(ep);
        ew = wave_sum(ew);
        if (lane == 0) { a.spart[2 * tile] = ep; a.spart[2 * tile + 1] = ew; }
    } else {
        double qphi = 0.0, qdt = 0.0, qdb = 0.0;
        if (active) {
            const int i = a.sidx[t];
            const double qi = me.w * d.pref;
            double4 *o = a.parts > 1 ? a.freal_s + (int64_t)blockIdx.y * a.n_total : a.freal;
            o[i] = make_double4(qi * fx, qi * fy, qi * fz, d.pref * phi);
            qphi = qi * phi;
            if (DG) { qdt = qi * dpt; qdb = qi * dpb; }
        }
        // per-tile sums (a tile never straddles two systems)
        qphi = wave_sum(qphi);
        if (DG) { qdt = wave_sum(qdt); qdb = wave_sum(qdb); }
        if (lane == 0) {
            double *o = a.parts > 1 ? a.rpart_s + 3 * ((int64_t)blockIdx.y * a.n_waves + tile) : a.rpart + 3 * tile;
            o[0] = qphi;
            o[1] = qdt;
            o[2] = qdb;
        }
    }
}

template <TileKind KIND>
static TileArgs tile_args(rbe2d_ctx *h) {
    TileArgs r{};
    r.src = h->w.sorted; r.sidx = h->w.sidx; r.start = h->w.start;
    r.sys = h->w.sys; r.fam = h->w.fam; r.lay = h->w.lay; r.n_sys = h->n_sys; r.n_total = (int)h->n_total; r.n_waves = h->n_swaves;
    r.freal = h->w.freal; r.rpart = h->w.rpart; r.freal_s = h->w.freal_s; r.rpart_s = h->w.rpart_s; r.spart = h->w.spart;
    // Too few tiles to fill the chip: 4 or 2 waves share one, and up to 384 tiles
    // as many blocks of 4 waves as the chip holds at once (3 waves per SIMD of
    // 256 CUs): a lone wave of a SIMD is bound by its chain of instructions.
    // Force calls with one block of 12 (to 256 tiles) or 4 waves | with parts:
    // 4000 ions 66 | 56 and 75 | 58 us, 10000 81 | 75, 20000 101 | 83 and 129 |
    // 100.  Two or three parts of 385 to 768 tiles change less than 4 % either
    // way.  64000 ions: 2 waves 160, 4 waves 166; 120000: 2 waves 237, 1 wave 272.
    int n = h->n_swaves <= 768 ? 2 : h->n_swaves <= 2048 ? 1 : 0;
    r.parts = 1;
    if (KIND == kWca) {
        // little work per tile: up to 12 waves of one block
        if (h->n_swaves <= 256) { r.wpt = kMaxTileWaves; return r; }
    } else {
        if (n == 2) n = 3;
        if (h->force_rsplit) n = h->force_rsplit - 1;
        else if (h->tuned_now && h->tune.rsplit) n = h->tune.rsplit - 1;
        if (n >= 3) r.parts = tile_parts(h->n_swaves);
    }
    r.wpt = 1 << std::min(n, 2);
    return r;
}

template <TileKind KIND, bool DG>
static void launch_tile(TileArgs r, const AssembleArgs *as, hipStream_t s) {
    const int waves = std::max(4, r.wpt);            // per block
    const int per_block = waves / r.wpt;
    r.nblocks = (r.n_waves + per_block - 1) / per_block;
    const int nch = 8 * kTileChunks;
    r.nbx = (r.nblocks + nch - 1) / nch * nch;
    const int bytes = waves * TileLds<DG>::kWaveBytes;
    if constexpr (KIND == kErfc) {
        if (as) {
            const int row = waves * r.parts;
            hipLaunchKernelGGL((k_tile<KIND, DG, true>), dim3(r.nbx + (as->items() + row - 1) / row, r.parts), dim3(waves * kWave), bytes, s, r, *as);
            return;
        }
    }
    hipLaunchKernelGGL((k_tile<KIND, DG, false>), dim3(r.nbx, r.parts), dim3(waves * kWave), bytes, s, r, AssembleArgs());
}

void launch_tile_pairs(rbe2d_ctx *h, bool want_dg, const AssembleArgs *as, hipStream_t s) {
    const TileArgs r = tile_args<kErfc>(h);
    h->real_parts = r.parts;
    h->real_stride = h->n_swaves;
    prof_begin(h, 4, s);
    if (want_dg) launch_tile<kErfc, true>(r, as, s);
    else launch_tile<kErfc, false>(r, as, s);
    prof_end(h, 4, s);
}

// ---------------------------------------------------------------------------
// Short-range forces of the MD (purely repulsive shifted-truncated LJ between
// ions and against the walls): the tiles of the pair sum with the LJ cutoff
// and no images, in FP64.  Forces are added to the caller's N x 3 forces, or in
// an MD step kept as one more part of the real-space forces: the step runs
// this launch beside the pair kernel's.  Per-tile energy sums go to spart.
// ---------------------------------------------------------------------------

// The same by one thread per target, over the runs of cells within the cutoff.
// On the FP32 pair kernel's fine cells (r_c / 6 along y) it scans 50 ions per
// target where a tile, 60 units long on the 1e6-ion slab, takes 600 candidates;
// with few targets its chain of gathers is what a launch lasts.  Langevin steps
// with it | with tiles: 1e6 ions 1.28 | 1.48 ms, 60000 168 | 192 us, 30000 130 |
// 134, 20000 117 | 113.
struct ScanArgs {
    const double4 *src;
    const int *sidx, *scell, *start;
    const SysDesc *sys;
    Layout lay;
    int n_sys, n_waves;
    MdExtra mx;
    double *F;                  // added to when set, else written to freal
    double4 *freal;
    double *spart;
};
__global__ __launch_bounds__(kBlock) void k_short(ScanArgs a) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    const int r = __builtin_amdgcn_readfirstlane(find_sys(a.lay.sbase, a.n_sys, t & ~(kWave - 1)));
    const SysDesc d = a.sys[r];
    const int shift = a.lay.sbase[r] - a.lay.off[r];
    const bool active = t - a.lay.sbase[r] < a.lay.off[r + 1] - a.lay.off[r];
    double fx = 0, fy = 0, fz = 0, ep = 0, ew = 0;
    if (active) {
        const double4 me = a.src[t];
        const int cid = a.scell[t];
        const int cy = cid % d.ncy, cx = (cid / d.ncy) % d.ncx;
        if (a.mx.eps != 0.0) {
            // cell ranges within the cutoff, with a 1e-9 margin (cells were
            // assigned by division); a small box searches each column or row once
            const double rc = sqrt(a.mx.rc2) * (1.0 + 1e-9);
            const int rx = (int)ceil(rc / d.hx), ry = (int)ceil(rc / d.hy);
            const bool allx = d.ncx <= 2 * rx, ally = d.ncy <= 2 * ry;
            const double xrel = me.x - cx * d.hx, yrel = me.y - cy * d.hy;
            const int x0 = allx ? 0 : cx + (int)floor((xrel - rc) * d.inv_hx);
            const int x1 = allx ? d.ncx - 1 : cx + (int)floor((xrel + rc) * d.inv_hx);
            const int y0 = ally ? 0 : cy + (int)floor((yrel - rc) * d.inv_hy);
            const int y1 = ally ? d.ncy - 1 : cy + (int)floor((yrel + rc) * d.inv_hy);
            const int z0 = max(0, (int)floor((me.z - rc) * d.inv_hz));
            const int z1 = min(d.ncz - 1, (int)floor((me.z + rc) * d.inv_hz));
            const int *start = a.start + d.cbase;
            for (int lz = z0; lz <= z1; lz++)
                for (int ix = x0; ix <= x1; ix++) {
                    const int row = (lz * d.ncx + (ix % d.ncx + d.ncx) % d.ncx) * d.ncy;
                    // along y: one run of cells, or two where it wraps
                    for (int part = 0; part < 2; part++) {
                        int ya = y0, yb = y1;
                        if (!ally) {
                            if (part == 0) { ya = max(y0, 0); yb = min(y1, d.ncy - 1); }
                            else if (y0 < 0) { ya = y0 + d.ncy; yb = d.ncy - 1; }
                            else if (y1 >= d.ncy) { ya = 0; yb = y1 - d.ncy; }
                            else break;
                        } else if (part == 1) {
                            break;
                        }
                        if (ya > yb) continue;
                        const int b = start[row + ya] + shift, e = start[row + yb + 1] + shift;
                        for (int j = b; j < e; j++) {
                            if (j == t) continue;
                            const double4 sj = a.src[j];
                            double dx = me.x - sj.x, dy = me.y - sj.y;
                            dx -= d.Lx * rint(dx * d.inv_Lx);
                            dy -= d.Ly * rint(dy * d.inv_Ly);
                            const double dz = me.z - sj.z;
                            const double r2 = dx * dx + dy * dy + dz * dz;
                            if (r2 < a.mx.rc2) {
                                double rf;
                                ep += 0.5 * lj_rep(a.mx.sig2 / r2, a.mx.eps, &rf);
                                fx += rf / r2 * dx; fy += rf / r2 * dy; fz += rf / r2 * dz;
                            }
                        }
                    }
                }
        }
        ew = wall_terms(a.mx, d, me.z, &fz);
        const int i = a.sidx[t];
        if (a.F) {
            double *o = a.F + (int64_t)3 * i;
            o[0] += fx; o[1] += fy; o[2] += fz;
        } else {
            a.freal[i] = make_double4(fx, fy, fz, 0.0);
        }
    }
    ep = wave_sum(ep);
    ew = wave_sum(ew);
    if ((threadIdx.x & (kWave - 1)) == 0 && t / kWave < a.n_waves) {
        a.spart[2 * (t / kWave)] = ep;
        a.spart[2 * (t / kWave) + 1] = ew;
    }
}

// per-system sums of the wave energies, fixed order
__global__ __launch_bounds__(kBlock) void k_short_energy(const double *spart, Layout lay, double *energy) {
    __shared__ double sh[kBlock / 64];
    const int r = blockIdx.x;
    double ep = 0, ew = 0;
    for (int wv = lay.sbase[r] / kWave + threadIdx.x; wv < lay.sbase[r + 1] / kWave; wv += kBlock) {
        ep += spart[2 * wv];
        ew += spart[2 * wv + 1];
    }
    ep = block_sum(ep, sh);
    ew = block_sum(ew, sh);
    if (threadIdx.x == 0) {
        energy[2 * r] = ep;
        energy[2 * r + 1] = ew;
    }
}

hipError_t launch_short(rbe2d_ctx *h, const MdExtra &mx, double *F, double *energy, hipStream_t s) {
    prof_begin(h, 9, s);
    if (h->n_total > 0 && mx.short_on()) {
        h->short_part = !F;
        if (h->precision == RBE2D_PREC_FP32_PHASE && h->n_total > kShortTiles32) {
            ScanArgs a;
            a.src = h->w.sorted; a.sidx = h->w.sidx; a.scell = h->w.scell; a.start = h->w.start;
            a.sys = h->w.sys; a.lay = h->w.lay; a.n_sys = h->n_sys; a.n_waves = h->n_swaves;
            a.mx = mx; a.F = F; a.freal = h->w.fshort; a.spart = h->w.spart;
            hipLaunchKernelGGL(k_short, dim3((h->n_swaves * kWave + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
        } else {
            TileArgs a = tile_args<kWca>(h);
            a.mx = mx; a.F = F; a.freal = h->w.fshort;
            launch_tile<kWca, false>(a, nullptr, s);
        }
    }
    hipError_t e = hipGetLastError();
    if (energy && e == hipSuccess) {
        if (h->n_total > 0 && mx.short_on()) {
            hipLaunchKernelGGL(k_short_energy, dim3(h->n_sys), dim3(kBlock), 0, s, h->w.spart, h->w.lay, energy);
            e = hipGetLastError();
        } else {
            e = launch_fill(energy, (int64_t)h->n_sys * 2 * sizeof(double), s);
        }
    }
    prof_end(h, 9, s);
    return e;
}

}  // namespace rbe2d
