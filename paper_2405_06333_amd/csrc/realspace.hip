// Real-space half of RBE2D on gfx950 (Eq. (3.12)): a cell list over each
// slab built by counting sort with a deterministic in-cell order, and the
// erfc pair sum over real charges and truncated image charges within r_c for
// FP32 phases (tiles.hip has the FP64 one).  All systems of a handle share
// one sort (their cells are numbered consecutively) and one launch of the
// pair kernel.
//
// Images are never materialised: the order-l image of source j is at the
// same distance from target i as the real source j is from a transformed
// target (x_i, y_i, sz z_i + cz) -- a reflection for odd l, a shift for even
// l -- so every image family is another cell search around the transformed
// target, done only when that point lies within r_c of the slab.
#include <algorithm>

#include "devmath.h"
#include "energy.h"
#include "erfcx_fit.h"
#include "kspace_dev.h"
#include "rbe2d_internal.h"

// Compile-time parameters of the FP32 pair kernel (measured best on the
// 1e6-ion slab: 16-entry rings halve the occupancy, batches of 2 loads leave
// latency exposed, the drain threshold hardly matters).  Register cap: the
// double-buffered scan of paired columns fits 4 waves per SIMD without
// spills (122 VGPRs); at 5 waves it spills and is 5 % slower, uncapped at 3
// waves slower still.
#ifndef RBE2D_REAL_U32
#define RBE2D_REAL_U32 4      // source loads per batch (two batches in flight per lane)
#endif
#ifndef RBE2D_RING_Q
#define RBE2D_RING_Q 8        // ring entries per lane (a power of two)
#endif
#ifndef RBE2D_ROUND_MIN
#define RBE2D_ROUND_MIN 40    // keep draining while this many lanes hold pairs
#endif
#ifndef RBE2D_REAL_CHUNKS
#define RBE2D_REAL_CHUNKS 8   // contiguous target chunks per XCD
#endif
#ifndef RBE2D_REAL_WAVES32
#define RBE2D_REAL_WAVES32 4  // FP32 pair kernel: waves per SIMD its register budget must allow
#endif

namespace rbe2d {

__global__ void k_fill(uint32_t *p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

hipError_t launch_fill(void *p, int64_t nbytes, hipStream_t s) {
    const int64_t n = nbytes / 4;
    if (n > 0) hipLaunchKernelGGL(k_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (uint32_t *)p, n);
    return hipGetLastError();
}

struct CellArgs {
    const double *pos, *q;
    const SysDesc *sys;
    Layout lay;
    int n_sys, n_total, ncells;
    int *cell, *slot, *count, *start, *sidx, *scell;
    int2 *tmp;      // unordered cell lists: (caller index, global cell)
    int n_waves;    // padded sorted positions / 64 (the rank pass runs one wave per system chunk)
    // set when the MD pass that moved the particles (and counted them) also
    // wrote their k-space records on this stream: the rank pass reads those
    // (one aligned record per particle) instead of positions and charges
    const float4 *p32;
    const double4 *p64;
    double4 *sorted;        // (x wrapped, y wrapped, z, q)
    uint4 *src16;           // written (with scell) when set: FP32 pair kernel
};

// position -> 32-bit fixed point; the wrap of 2^32 is the period (x, y)
__device__ __forceinline__ uint32_t to_fixed(double v, double scale) {
    return (uint32_t)(unsigned long long)llrint(v * scale);
}

__global__ __launch_bounds__(kBlock) void k_cell_count(CellArgs a) {
    const int g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= a.n_total) return;
    const int r = find_sys(a.lay.off, a.n_sys, g);
    const SysDesc &d = a.sys[r];
    const int c = d.cbase + cell_of(a.pos[3 * (int64_t)g], a.pos[3 * (int64_t)g + 1], a.pos[3 * (int64_t)g + 2], d);
    a.cell[g] = c;
    a.slot[g] = atomicAdd(&a.count[c], 1);
}

// exclusive scan of count[0..ncells) into start[0..ncells]: each block of 4096
// cells adds the cells before it to the scan of its own.  Up to kScanDirect
// blocks it reads their counts itself; beyond, a launch of its own leaves the
// blocks' totals (at most a few hundred).  The scatter clears the counts for
// the next build.  Integer sums: the order does not matter.
constexpr int kScanPer = 16;                      // cells per thread
constexpr int kScanCells = kBlock * kScanPer;     // cells per scan block
constexpr int kScanDirect = 8;                    // (2 or 32: the same within 1 %)

__device__ __forceinline__ void load_counts(const int *count, int n, int c0, int (&v)[kScanPer]) {
    if (c0 + kScanPer <= n && (c0 & 3) == 0) {
        const int4 *p = reinterpret_cast<const int4 *>(count + c0);
#pragma unroll
        for (int k = 0; k < kScanPer / 4; k++) {
            const int4 w = p[k];
            v[4 * k] = w.x; v[4 * k + 1] = w.y; v[4 * k + 2] = w.z; v[4 * k + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < kScanPer; k++) v[k] = c0 + k < n ? count[c0 + k] : 0;
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_totals(const int *count, int n, int *btot) {
    __shared__ int sh[kBlock / 64];
    int v[kScanPer];
    load_counts(count, n, blockIdx.x * kScanCells + threadIdx.x * kScanPer, v);
    int t = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; k++) t += v[k];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        int b = 0;
        for (int w = 0; w < kBlock / 64; w++) b += sh[w];
        btot[blockIdx.x] = b;
    }
}

// btot null: the cells before this block from their counts
__global__ __launch_bounds__(kBlock) void k_scan_apply(const int *count, int n, const int *btot, int *start) {
    __shared__ int sh_wave[kBlock / 64], sh_before[kBlock / 64];
    __shared__ int sh_base;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (!btot) {
        int b = 0;
        for (int k = 0; k < (int)blockIdx.x; k++) {
            int u[kScanPer];
            load_counts(count, n, k * kScanCells + threadIdx.x * kScanPer, u);
#pragma unroll
            for (int c = 0; c < kScanPer; c++) b += u[c];
        }
        b = wave_sum(b);
        if (lane == 0) sh_before[wid] = b;
    } else if (wid == 0) {
        // cells before this block: the totals of the blocks before it
        int b = 0;
        for (int k = lane; k < (int)blockIdx.x; k += 64) b += btot[k];
        b = wave_sum(b);
        if (lane == 0) sh_base = b;
    }
    const int c0 = blockIdx.x * kScanCells + threadIdx.x * kScanPer;
    int v[kScanPer];
    load_counts(count, n, c0, v);
    int t = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; k++) t += v[k];
    // inclusive scan of the thread totals over the wave, then over the waves
    int incl = t;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) sh_wave[wid] = incl;
    __syncthreads();
    int before = 0;
    if (btot) before = sh_base;
    else
        for (int w = 0; w < kBlock / 64; w++) before += sh_before[w];
    for (int w = 0; w < wid; w++) before += sh_wave[w];
    int run = before + incl - t;
#pragma unroll
    for (int k = 0; k < kScanPer; k++) {
        const int c = c0 + k;
        if (c < n) {
            start[c] = run;
        }
        run += v[k];
        if (c == n - 1) start[n] = run;
    }
}

__global__ __launch_bounds__(kBlock) void k_cell_scatter(CellArgs a) {
    const int g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= a.n_total) return;
    const int c = a.cell[g];
    a.tmp[a.start[c] + a.slot[g]] = make_int2(g, c);
    a.count[c] = 0;       // the next build counts from zero
}

// Particle gc.x of cell gc.y, whose members are at positions [b, e) of the
// unordered cell lists: its position within the cell = number of members with
// a smaller caller index, and its records there.
template <typename Tmp>
__device__ __forceinline__ void place_particle(const CellArgs &a, const SysDesc &d, int r, int2 gc, int b, int e,
                                               Tmp tmp_index) {
    const int g = gc.x, c = gc.y;
    int rank = 0;
    for (int k = b; k < e; k++) rank += tmp_index(k) < g;
    const int s = b + rank + (a.lay.sbase[r] - a.lay.off[r]);
    double xw, yw, z, qg;
    if (a.p32 || a.p64) {
        // the particle's k-space record: fractional x, y (wrapped) and z / L_z,
        // split hi + lo in FP32 (46 significant bits) or exact in FP64, and q
        // (FP32 in the FP32 records, as the FP32 pair kernel uses it)
        const int64_t ii = (int64_t)a.lay.pbase[r] + (g - a.lay.off[r]);
        double fx, fy, fz;
        if (a.p32) {
            const float4 u = a.p32[2 * ii], v = a.p32[2 * ii + 1];
            fx = (double)u.x + (double)u.y; fy = (double)u.z + (double)u.w; fz = (double)v.x + (double)v.y;
            qg = (double)v.z;
        } else {
            const double4 u = a.p64[ii];
            fx = u.x; fy = u.y; fz = u.z; qg = u.w;
        }
        xw = fx * d.Lx; yw = fy * d.Ly; z = fz * d.Lz;
    } else {
        xw = wrapped(a.pos[3 * (int64_t)g], d.Lx);
        yw = wrapped(a.pos[3 * (int64_t)g + 1], d.Ly);
        z = a.pos[3 * (int64_t)g + 2];
        qg = a.q[g];
    }
    a.sorted[s] = make_double4(xw, yw, z, qg);
    a.sidx[s] = g;
    if (a.src16) {
        a.scell[s] = c - d.cbase;   // the cell it was counted in
        // z clamped into the frame (z outside (0, H) is flagged by prep)
        const double zc = fmin(fmax(z, -d.rc), d.H + d.rc);
        a.src16[s] = make_uint4(to_fixed(xw, d.fxs), to_fixed(yw, d.fys), to_fixed(zc + d.zoff, d.fzs),
                                __float_as_uint((float)qg));
    }
}

// SF: the structure factors of the call (FP32 or FP64) are further blocks of
// the cell-list launch.  On one stream they wait for each other otherwise, with
// most of the chip idle: 500 ions, 5 + 5 us.
enum SfKind { kNoSf, kSf32, kSf64 };
template <SfKind SF>
struct SfRide {
    static constexpr int kLds = SF == kNoSf ? 1 : SF == kSf32 ? sizeof(SfLds32<kKChunk32>) : sizeof(SfLds64<kKChunk64>);
    // part `b` of the structure factors by kBlock threads (past the last: the last once more)
    static __device__ __forceinline__ void run(const SfArgs &a, int b, int tid, void *lds) {
        const int nkc = a.P_pad / (SF == kSf32 ? kKChunk32 : kKChunk64);
        b = min(b, a.n_tiles * nkc - 1);
        const TileChunk tc{b / nkc, b % nkc};
        if constexpr (SF == kSf32)
            sf32_block<kKChunk32, true>(a.p32, a.kn32, a.tbase, a.n_sys, a.per, a.P_pad, a.part, tc, tid,
                                        ((SfLds32<kKChunk32> *)lds)->sh);
        if constexpr (SF == kSf64) {
            SfLds64<kKChunk64> *l = (SfLds64<kKChunk64> *)lds;
            sf64_block<kKChunk64, true>(a.p64, a.kn64, a.tbase, a.n_sys, a.per, a.P_pad, a.part, tc, tid, l->sh, l->tab);
        }
    }
    static int parts(const SfArgs &a) { return a.n_tiles * (a.P_pad / (SF == kSf32 ? kKChunk32 : kKChunk64)); }
};

// Sorted positions are padded per system to whole waves.  One thread per
// padded sorted position, so a wave belongs to one system (its constants
// are scalar loads); the thread takes slot j of the unordered cell lists
// (tmp), gathers the particle it holds and writes its record within the
// same cell, so the stores of a wave stay within a few neighbouring cells.
template <SfKind SF>
__global__ __launch_bounds__(kBlock) void k_cell_rank(CellArgs a, SfArgs sf, int n_sf) {
    if constexpr (SF != kNoSf) {
        __shared__ __align__(16) unsigned char lds[SfRide<SF>::kLds];
        if ((int)blockIdx.x < n_sf) {
            SfRide<SF>::run(sf, blockIdx.x, threadIdx.x, lds);
            return;
        }
    }
    const int t = (blockIdx.x - n_sf) * kBlock + threadIdx.x;
    if (t >= a.n_waves * kWave) return;
    const int r = __builtin_amdgcn_readfirstlane(find_sys(a.lay.sbase, a.n_sys, t & ~(kWave - 1)));
    const SysDesc d = a.sys[r];   // a copy: wave-uniform values in scalar registers
    const int j = t - a.lay.sbase[r] + a.lay.off[r];   // position in the unpadded cell lists
    if (j >= a.lay.off[r + 1]) return;                   // padding of this system
    const int2 gc = a.tmp[j];
    place_particle(a, d, r, gc, a.start[gc.y], a.start[gc.y + 1], [&](int k) { return a.tmp[k].x; });
}

// The whole build after the count in one launch, one block per system: a scan
// of the system's cells (its first position is its particle offset), their
// lists and the ordered records, through LDS, which has to hold the cells'
// starts and the lists.  It takes the place of four launches of 5 to 6 us.
// Beyond kSmallN particles in a system one block is slower than they are: a
// force call of 10000 ions takes 109 us with it and 90 without, 16 slabs of
// 300 to 3200 ions 95 with it and 101 without.
constexpr int kSmallThreads = 1024;
constexpr size_t kSmallLds = 60 << 10;
constexpr int kSmallN = 4096;
// More than kManySystems systems: blocks of kBlock threads up to kNarrowN
// particles each, since several share a CU then and most threads of 1024 have
// nothing to do; and from kTinySystems systems of up to kTinyN on, with nothing
// riding along, the four launches, which take less of the chip from the k-space
// chain beside them.  Velocity-Verlet steps with 1024 | 256 threads | four
// launches: 16384 slabs of 8 ions FP32 1054 | 954 | 950 us, 1024 of 16 116 | 119 |
// 109, 256 of 100 108 | 108 | 103, 200 of 16 59 | 59 | 69, 1024 of 200 325 | 244 |
// 343, 300 of 1000 340 | 344 | 373.
constexpr int kManySystems = 128, kNarrowN = 512, kTinySystems = 256, kTinyN = 128;
template <SfKind SF>
__global__ __launch_bounds__(kSmallThreads) void k_cells_small(CellArgs a, SfArgs sf) {
    extern __shared__ __align__(16) int lds[];
    __shared__ int sh[kSmallThreads / kWave];
    const int r = blockIdx.x;
    if constexpr (SF != kNoSf) {
        if (r >= a.n_sys) {
            const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock);
            SfRide<SF>::run(sf, (r - a.n_sys) * (int)(blockDim.x / kBlock) + sub, threadIdx.x % kBlock,
                            (char *)lds + sub * SfRide<SF>::kLds);
            return;
        }
    }
    const int nt = blockDim.x;
    const SysDesc &d = a.sys[r];
    const int off = a.lay.off[r], N = a.lay.off[r + 1] - off;
    const int c0 = d.cbase, nc = d.ncx * d.ncy * d.ncz;
    int *start = lds;                                             // positions within the system
    int *tmp = lds + nc + 1;                                      // cell lists: indices within the system
    const int per = (nc + nt - 1) / nt;
    const int lo = min(nc, (int)threadIdx.x * per), hi = min(nc, lo + per);
    for (int c = threadIdx.x; c < nc; c += nt) {
        start[c] = a.count[c0 + c];
        a.count[c0 + c] = 0;                                      // the next build counts from zero
    }
    __syncthreads();
    int t = 0;
    for (int c = lo; c < hi; c++) t += start[c];
    int run = block_scan(t, sh);
    for (int c = lo; c < hi; c++) {
        const int v = start[c];
        start[c] = run;
        run += v;
    }
    if (threadIdx.x == 0) start[nc] = N;
    __syncthreads();
    // (the next system's first start equals this one's end)
    for (int c = threadIdx.x; c < nc; c += nt) a.start[c0 + c] = off + start[c];
    if (r == a.n_sys - 1 && threadIdx.x == 0) a.start[c0 + nc] = off + N;
    for (int i = threadIdx.x; i < N; i += nt) {
        const int c = a.cell[off + i];
        tmp[start[c - c0] + a.slot[off + i]] = i;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < N; j += nt) {
        const int g = off + tmp[j], c = a.cell[g];
        place_particle(a, d, r, make_int2(g, c), off + start[c - c0], off + start[c - c0 + 1],
                       [&](int k) { return off + tmp[k - off]; });
    }
}

struct RealArgs {
    const double4 *src;         // sorted sources: (x wrapped, y wrapped, z, q)
    const uint4 *src16;         // the same in fixed point
    const int *sidx, *scell, *start;
    const SysDesc *sys;
    const Family *fam;          // kMaxFamilies per system
    Layout lay;
    int n_sys, n_waves;         // n_waves: padded real-space waves of all systems
    int nblocks;                // logical blocks (the grid is rounded up to 8 * RBE2D_REAL_CHUNKS chunks)
    int nbx;                    // ASM: blocks per grid row that sum pairs
    double4 *freal;
    double *rpart;              // per wave
    int nsplit;                 // > 1: block row y handles x-columns y, y + nsplit, ... of every target
    int64_t split_stride;       // targets per split in the partial outputs
    int rsplit_stride;          // waves per split in the partial wave sums
    double4 *freal_s;
    double *rpart_s;
};

// Constants of the FP32 pair terms in the units of the displacements: with
// displacements in units u (r = u rq), ec and fs below come out as u erfc(a r)/r
// and u^3 [erfc(a r)/r + 2a/sqrt(pi) e^{-a^2 r^2}]/r^2; the sums are rescaled
// by 1/u and 1/u^2 when they are folded into FP64.
struct PairConst32 {
    float ce;    // -a^2 u^2 log2(e): exp(-a^2 r^2) = 2^(ce rq^2)
    float cpx;   // p a u: the fit's argument p a r = cpx rq
    float c2a;   // 2a/sqrt(pi) u
    double fscale, pscale;   // 1/u^2 (forces), 1/u (potential)
    __device__ PairConst32(double alpha, double u)
        : ce(uniform((float)(-alpha * alpha * u * u * 1.4426950408889634))),
          cpx(uniform((float)(RBE2D_ERFCX_P * alpha * u))), c2a(uniform((float)(1.1283791670955126 * alpha * u))),
          fscale(uniform(1.0 / (u * u))), pscale(uniform(1.0 / u)) {}
};

// erfc(a r)/r (ec) and the radial force factor fs = [erfc(a r)/r + 2a/sqrt(pi)
// e^{-a^2 r^2}]/r^2 from rq^2, both in the units of PairConst32; erfc(x) =
// e^{-x^2} t P7(t), t = 1/(1 + p x), the fitted erfcx.
__device__ __forceinline__ void pair_terms(float r2, const PairConst32 &c, float *ec, float *fs) {
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float e = __builtin_amdgcn_exp2f(c.ce * r2);
    const float t = __builtin_amdgcn_rcpf(fmaf(c.cpx, r2 * rinv, 1.0f));
    float p = rbe2d_erfcx_a[RBE2D_ERFCX_DEG - 1];
#pragma unroll
    for (int k = RBE2D_ERFCX_DEG - 2; k >= 0; k--) p = fmaf(p, t, rbe2d_erfcx_a[k]);
    const float v = e * p * t * rinv;
    *ec = v;
    *fs = fmaf(c.c2a, e, v) * (rinv * rinv);
}

// ---------------------------------------------------------------------------
// Queues of accepted pairs.  The scan appends pairs (displacement from the
// source to the target, source charge); evaluating erfc/exp for them is
// deferred so that it runs with as many lanes busy as possible.  Both give
// the sums of the queued pairs' force and potential terms in FP64.
// ---------------------------------------------------------------------------

// Per-target FP64 sums over all image families.  Each drain's sums are
// added with the current family's weights: w for x, y and the potential,
// w * zsign for z (the image height moves against the target's for odd
// orders), dw / dgamma for the gamma derivatives of the potential; `scale`
// converts force sums kept in other units.
template <bool DG>
struct TargetSums {
    double fx = 0, fy = 0, fz = 0, phi = 0, dpt = 0, dpb = 0;
    double wxy = 1, wz = 1, wp = 1, wt = 0, wb = 0;
    // fscale, pscale: unit conversions of the force and potential sums
    __device__ void family(double w, double zsign, double dwt, double dwb, double fscale, double pscale) {
        wxy = uniform(w * fscale); wz = uniform(w * zsign * fscale); wp = uniform(w * pscale);
        if (DG) { wt = uniform(dwt * pscale); wb = uniform(dwb * pscale); }
    }
    __device__ void add(double sx, double sy, double sz, double sp) {
        fx = fma(sx, wxy, fx); fy = fma(sy, wxy, fy); fz = fma(sz, wz, fz); phi = fma(sp, wp, phi);
        if (DG) { dpt = fma(sp, wt, dpt); dpb = fma(sp, wb, dpb); }
    }
};

// popcount of a wave mask as two 32-bit halves (scalar instructions only)
__device__ __forceinline__ int busy_lanes(uint64_t m) {
    return __builtin_popcount((uint32_t)m) + __builtin_popcount((uint32_t)(m >> 32));
}

// FP32 kernel: a ring of Q entries per lane.  A round evaluates the oldest
// entry of every lane that holds one; the FP32 sums of a drain (at most Q
// pairs per lane) are folded into FP64.  Cheap routing (every result stays in
// its lane) at the price of idle lanes in the rounds.  The lane's read and
// write positions are byte counters into the slot-major rings (one 16-byte
// entry per thread and slot), masked only to form an address; their
// difference is the fill.  ISO: entries hold displacements in units of the
// isotropic fixed-point frame and the pair terms are evaluated in those units.
template <int Q, int U, bool ISO, bool DG>
struct LaneRings : TargetSums<DG> {
    static constexpr int kRoundMin = RBE2D_ROUND_MIN;   // keep draining while this many lanes hold pairs
    static constexpr uint32_t kSlot = kBlock * (uint32_t)sizeof(float4);
    static constexpr uint32_t kMask = Q * kSlot - 1;    // Q * kSlot is a power of two
    static constexpr uint32_t kRoom = (Q - U) * kSlot;  // fill beyond which U more pushes may not fit
    unsigned char *base;
    uint32_t wpos, rpos;   // unsigned: the counters may wrap, their difference stays exact
    PairConst32 pc;
    float sx = 0, sy = 0, sz = 0, sp = 0;
    __device__ LaneRings(unsigned char *b, int t, const SysDesc &d)
        : base(b), wpos((uint32_t)t * (uint32_t)sizeof(float4)), rpos(wpos), pc(d.alpha, ISO ? d.ud : 1.0) {}
    __device__ void family(double w, double zsign, double dwt, double dwb) {
        TargetSums<DG>::family(w, zsign, dwt, dwb, pc.fscale, pc.pscale);
    }
    __device__ void push(bool acc, float dx, float dy, float dz, float qs) {
        if (acc) {
            const uint32_t at = wpos & kMask;
            wpos += kSlot;
            *reinterpret_cast<float4 *>(base + at) = make_float4(dx, dy, dz, qs);
        }
    }
    // without a branch: rejected pairs go to the slot behind the ring
    __device__ void push_masked(bool acc, float dx, float dy, float dz, float qs) {
        const uint32_t at = acc ? wpos & kMask : (uint32_t)(threadIdx.x * sizeof(float4)) + Q * kSlot;
        *reinterpret_cast<float4 *>(base + at) = make_float4(dx, dy, dz, qs);
        wpos += acc ? kSlot : 0u;
    }
    __device__ bool full() const { return __ballot(wpos - rpos > kRoom) != 0; }
    // one round: evaluate the oldest entry of every lane with fill f > 0
    __device__ void round(uint32_t f) {
        if (f != 0) {
            const float4 e = *reinterpret_cast<const float4 *>(base + (rpos & kMask));
            rpos += kSlot;
            const float r2 = e.x * e.x + e.y * e.y + e.z * e.z;
            float ec, fs;
            pair_terms(r2, pc, &ec, &fs);
            const float qf = e.w * fs;
            sx += qf * e.x; sy += qf * e.y; sz += qf * e.z; sp += e.w * ec;
        }
    }
    __device__ void fold() {
        this->add((double)sx, (double)sy, (double)sz, (double)sp);
        sx = sy = sz = sp = 0;
    }
    // make room for U more pairs per lane: rounds while a lane could
    // overflow or while enough lanes hold pairs
    __device__ void drain() {
        uint32_t f = wpos - rpos;
        do {
            round(f);
            f = wpos - rpos;
        } while (__ballot(f > kRoom) != 0 || busy_lanes(__ballot(f != 0)) >= kRoundMin);
        fold();
    }
    __device__ void flush() {
        uint32_t f = wpos - rpos;
        while (__ballot(f != 0) != 0) {
            round(f);
            f = wpos - rpos;
        }
        fold();
    }
};

// One thread per target, targets in cell order (z-layer slowest, then x,
// then y), so the lanes of a wave share a z-layer and see neighbour rows of
// similar length; every wave belongs to one system.  For each image family,
// each z-layer within r_c and each x-column, the sources lie in one
// contiguous run of cells along y (two runs where the range wraps around the
// periodic y boundary), culled to the y-extent the sphere of radius r_c
// allows in that layer and column.  Pairs within r_c are queued and their
// erfc/exp terms evaluated later in rounds (LaneRings, above).
// The sources are 16-byte fixed-point records: a displacement is an
// exact integer difference rounded once to FP32, so its error is one
// position quantum (period / 2^32); pairs so close that this would matter
// (the closest pairs dominate the force) are recomputed from the FP64
// records.  It evaluates erfc/exp and the per-drain partial sums in FP32 and
// accumulates the drains in FP64.  The order of every sum is fixed by the
// data, so the results are bitwise reproducible.
//
// SPLIT: too few targets to fill the chip.  1: block row y takes every
// nsplit-th column.  2, up to kFamilySplitMax targets: besides, block layer z
// takes one group of image families (0: the real charges); a wave is then
// nearly alone on its SIMD and bound by its own chain of instructions,
// branches above all: the candidates of a batch are tested without one, and
// the target itself is not sent through the FP64 geometry.  (Two rounds at a
// time, or two and four batches of sources in flight, took 4 to 10 % longer.)
// The FP32 sums are those of the same drains in every form.  3,000 ions, 300
// pairs each: 63 us instead of 99.  Whole force calls of 24,000 ions with
// 2 against 1: 93 against 111 and 125 against 160 us; of 64,000: 142 against
// 139 and 192 against 187.
//
// ASM: the per-k assembly of the call rides along (blocks from nbx on of each
// grid row), which on one stream waits for its end otherwise.
template <bool WANT_DG, bool ISO, int SPLIT, bool ASM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(SPLIT == 2 ? 2 : RBE2D_REAL_WAVES32, 8)))
void k_real(RealArgs a, AssembleArgs as) {
    constexpr bool FEW = SPLIT == 2;
    constexpr int U = RBE2D_REAL_U32;      // source loads in flight per lane, twice
    constexpr int kRingQ = RBE2D_RING_Q;   // ring entries per lane
    using Queue = LaneRings<kRingQ, U, ISO, WANT_DG>;
    __shared__ __align__(16) unsigned char lds[sizeof(float4) * (kRingQ + (FEW ? 1 : 0)) * kBlock];
    const double4 *src = a.src;
    const int tid = threadIdx.x;
    // Blocks are dealt round-robin to the 8 XCDs.  Each XCD runs C contiguous
    // chunks of targets (chunk k of XCD x is chunk 8k + x of the range), so
    // neighbouring cells share that XCD's L2, and the targets near the walls
    // (cell order is z-slowest; they search extra image families) are shared
    // by all XCDs instead of loading the first and last ones.
    const int nbx = ASM ? a.nbx : (int)gridDim.x;
    if constexpr (ASM) {
        if ((int)blockIdx.x >= nbx) {
            const int b = (((int)blockIdx.x - nbx) * gridDim.z + blockIdx.z) * gridDim.y + blockIdx.y;
            assemble_wave<WANT_DG>(as, b * (kBlock / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave),
                                   threadIdx.x % kWave);
            return;
        }
    }
    const int cs = (nbx >> 3) / RBE2D_REAL_CHUNKS;   // blocks per chunk
    const int j = (int)(blockIdx.x >> 3);
    const int lb = ((j / cs) * 8 + (int)(blockIdx.x & 7)) * cs + j % cs;
    if (lb >= a.nblocks) return;
    const int t = lb * kBlock + tid;
    // the system of this wave (system ranges are padded to whole waves)
    const int r = __builtin_amdgcn_readfirstlane(find_sys(a.lay.sbase, a.n_sys, t & ~(kWave - 1)));
    const SysDesc d = a.sys[r];   // a copy: loop-invariant values stay in registers
    const int shift = a.lay.sbase[r] - a.lay.off[r];    // unpadded -> padded sorted position
    const bool active = t - a.lay.sbase[r] < a.lay.off[r + 1] - a.lay.off[r];
    const Family *fams = a.fam + (int64_t)r * kMaxFamilies;
    const int *start = a.start + d.cbase;
    double4 me = make_double4(0.0, 0.0, 0.0, 0.0);
    int cid = 0;
    uint32_t xtf = 0, ytf = 0;   // target in fixed point
    if (active) {
        me = src[t];
        cid = a.scell[t];
        const uint4 m16 = a.src16[t];
        xtf = m16.x; ytf = m16.y;
    }
    const int cy = cid % d.ncy;
    const int cx = (cid / d.ncy) % d.ncx;
    const bool allx = d.ncx < 2 * d.reach + 1, ally = d.ncy < 2 * d.reach_y + 1;
    // Culling bounds are computed in FP32 with margins that cover its
    // rounding (and the division that assigned the cells): 1e-4 r_c^2 on the
    // squared y-extent, 1e-5 r_c on the extent.  They only decide which cells
    // are scanned; every candidate is then tested against r_c.
    const float yrel = (float)(me.y - cy * d.hy);   // y within the target's cell
    const float xrel = (float)(me.x - cx * d.hx);   // x within the target's cell
    const float hxf = (float)d.hx, inv_hyf = (float)d.inv_hy;
    const float rcm2 = (float)(d.rc2 * (1.0 + 1e-4));
    const float rmarg = (float)(1e-5 * d.rc);
    Queue qu(lds, tid, d);
    // claims all 128 registers a wave may hold at 4 waves per SIMD (the kernel
    // uses 119): waves of the force pass (32 registers) would join the four
    // otherwise and slow both, MD step of the 1e6-ion slab 1.25 instead of 1.22 ms
    if constexpr (!FEW) asm volatile("" ::: "v127");
    // with more than one layer of blocks: layer 0 the real charges, layers z >
    // 0 the families z, z + (layers - 1), ...
    const int fstep = FEW && gridDim.z > 1 ? (blockIdx.z == 0 ? kMaxFamilies + 1 : (int)gridDim.z - 1) : 1;
    for (int f = FEW ? (int)blockIdx.z : 0; f <= d.nfam; f += fstep) {
        double sz = 1.0, czs = 0.0, w = 1.0, zsign = 1.0, dwt = 0.0, dwb = 0.0;
        if (f > 0) {
            const Family fm = fams[f - 1];
            sz = fm.sz; czs = fm.cz; w = fm.w; zsign = fm.zsign; dwt = fm.dwt; dwb = fm.dwb;
        }
        const double tz = sz * me.z + czs;
        const bool fam_on = active && tz > -d.rc && tz < d.H_rc;
        if (__ballot(fam_on) == 0) continue;
        const uint32_t tzf = fam_on ? to_fixed(tz + d.zoff, d.fzs) : 0u;
        int lzlo = d.ncz, lzhi = -1;
        if (fam_on) {
            lzlo = max(0, (int)floor((tz - d.rc_lay) * d.inv_hz));
            lzhi = min(d.ncz - 1, (int)floor((tz + d.rc_lay) * d.inv_hz));
        }
        const int wzlo = wave_min(lzlo), wzhi = wave_max(lzhi);
        qu.family(w, zsign, dwt, dwb);
        // FP32: scan run A [jbA, jbA + lenA), then run B, for pairs within
        // r_c.  Each lane walks its two runs as one sequence: A's batches of U
        // (the last one padded), then B's.  The trip count is the wave
        // maximum, so drains always run with every lane; pairing the columns
        // on either side of the target's (one long where the other is short)
        // evens out the lanes' trip counts.  A lone run is B empty.  Loads are
        // issued U at a time, double-buffered: the next U records are in
        // flight while these are tested (and while a drain runs); without
        // the gamma derivatives the two buffers swap roles every batch (the
        // loop body is unrolled by two), so no records are copied between them.
        auto scan = [&](int jbA, int lenA, int jbB, int lenB) {
                const int c4a = (lenA + U - 1) / U * U;
                const int tot = c4a + lenB;
                const int maxtot = wave_max(tot);
                // loads from run B are clamped to min(m - c4a, lenB - 1): past a
                // run they stay within the padded arrays (jb + len - 1 + U - 1 <
                // capacity + 64) and are rejected
                const int lmB = max(lenB - 1, 0);
                auto rec = [&](int m0) { return m0 < c4a ? jbA + m0 : jbB + min(m0 - c4a, lmB); };
                // fixed-point displacements: exact integer differences (the
                // int32 wrap is the minimum image in x and y), one rounding
                // each to FP32; exact FP64 geometry for pairs within `near`
                const float rc2s = ISO ? d.rc2q : d.rc2f;
                const float near2s = ISO ? d.near2q : d.near2f;
                // exact FP64 displacement from sorted source js; false for zero
                // (the target itself in the direct family)
                auto near_pair = [&](int js, float &dx, float &dy, float &dz) {
                    const double4 s64 = src[js];
                    double ex = me.x - s64.x, ey = me.y - s64.y;
                    // the true displacement is below `near`, far from half a
                    // period, so rounding by the reciprocal finds the same image
                    ex -= d.Lx * rint(ex * d.inv_Lx);
                    ey -= d.Ly * rint(ey * d.inv_Ly);
                    const double ez = tz - s64.z;
                    const bool apart = ex != 0.0 || ey != 0.0 || ez != 0.0;
                    if (ISO) { ex *= d.fxs; ey *= d.fxs; }
                    dx = (float)ex; dy = (float)ey; dz = (float)(ISO ? ez * d.fxs : ez);
                    return apart;
                };
                auto body = [&](const uint4 (&sv)[U], int m0) {
                    if (qu.full()) qu.drain();
                    const bool inA = m0 < c4a;
                    const int lim = inA ? lenA : tot;          // candidates m < lim
                    if constexpr (FEW) {
                        // the four tests without a branch, one for the close
                        // pairs; the target itself is told by its index
                        const int j0 = jbA + m0;               // (no run B)
                        float dx[U], dy[U], dz[U];
                        bool acc[U], close[U], any = false;
#pragma unroll
                        for (int k = 0; k < U; k++) {
                            dx[k] = (float)(int)(xtf - sv[k].x);
                            dy[k] = (float)(int)(ytf - sv[k].y);
                            dz[k] = (float)(int)(tzf - sv[k].z);
                            if (!ISO) { dx[k] *= d.ux; dy[k] *= d.uy; dz[k] *= d.uz; }
                            const float r2 = fmaf(dx[k], dx[k], fmaf(dy[k], dy[k], dz[k] * dz[k]));
                            acc[k] = m0 + k < lenA && r2 < rc2s;
                            if (f == 0 && j0 + k == t) acc[k] = false;
                            close[k] = acc[k] && r2 < near2s;
                            any = any || close[k];
                        }
                        if (__ballot(any) != 0) {
#pragma unroll
                            for (int k = 0; k < U; k++)
                                if (close[k]) acc[k] = near_pair(j0 + k, dx[k], dy[k], dz[k]);
                        }
#pragma unroll
                        for (int k = 0; k < U; k++) qu.push_masked(acc[k], dx[k], dy[k], dz[k], __uint_as_float(sv[k].w));
                    } else {
#pragma unroll
                        for (int k = 0; k < U; k++) {
                            const int m = m0 + k;
                            float dx = (float)(int)(xtf - sv[k].x);
                            float dy = (float)(int)(ytf - sv[k].y);
                            float dz = (float)(int)(tzf - sv[k].z);
                            if (!ISO) { dx *= d.ux; dy *= d.uy; dz *= d.uz; }
                            const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
                            bool acc = m < lim && r2 < rc2s;
                            if (acc && r2 < near2s) acc = near_pair(inA ? jbA + m : jbB + (m - c4a), dx, dy, dz);
                            qu.push(acc, dx, dy, dz, __uint_as_float(sv[k].w));
                        }
                    }
                };
                if constexpr (FEW) {
                    // no prefetch: the chain of instructions is the longer one
                    for (int m0 = 0; m0 < maxtot; m0 += U) {
                        uint4 s[U];
                        const uint4 *pq = a.src16 + rec(m0);
#pragma unroll
                        for (int k = 0; k < U; k++) s[k] = pq[k];
                        body(s, m0);
                    }
                    return;
                }
                uint4 sa[U], sb[U];
                {
                    const uint4 *pq = a.src16 + rec(0);
#pragma unroll
                    for (int k = 0; k < U; k++) sa[k] = pq[k];
                }
                if constexpr (WANT_DG) {
                    // the gamma-derivative sums hold more registers: one loop
                    // body, the prefetched records copied into place
                    for (int m0 = 0; m0 < maxtot; m0 += U) {
                        if (m0 + U < maxtot) {
                            const uint4 *pq = a.src16 + rec(m0 + U);
#pragma unroll
                            for (int k = 0; k < U; k++) sb[k] = pq[k];
                        }
                        body(sa, m0);
#pragma unroll
                        for (int k = 0; k < U; k++) sa[k] = sb[k];
                    }
                } else {
                    for (int m0 = 0; m0 < maxtot; m0 += 2 * U) {
                        if (m0 + U < maxtot) {
                            const uint4 *pq = a.src16 + rec(m0 + U);
#pragma unroll
                            for (int k = 0; k < U; k++) sb[k] = pq[k];
                        }
                        body(sa, m0);
                        if (m0 + U >= maxtot) break;
                        if (m0 + 2 * U < maxtot) {
                            const uint4 *pq = a.src16 + rec(m0 + 2 * U);
#pragma unroll
                            for (int k = 0; k < U; k++) sa[k] = pq[k];
                        }
                        body(sb, m0 + U);
                    }
                }
        };
        // the runs of one column (cells along y within the sphere's extent
        // in this layer): [jb1, jb1 + len1) and, where the range wraps around
        // the periodic y boundary, [jb2, jb2 + len2)
        struct Runs {
            int jb1, len1, jb2, len2;
        };
        auto col_runs = [&](bool lay_on, int lz, float dzmin, int ox) {
            Runs R{0, 0, 0, 0};
            const int dxc = allx ? ox - cx : ox;       // column offset in cells
            int cxx = allx ? ox : cx + ox;
            if (!allx) cxx += cxx < 0 ? d.ncx : (cxx >= d.ncx ? -d.ncx : 0);
            float dxmin = 0.0f;
            if (!allx) dxmin = dxc > 0 ? dxc * hxf - xrel : (dxc < 0 ? xrel - (dxc + 1) * hxf : 0.0f);
            const float ye2 = rcm2 - dxmin * dxmin - dzmin * dzmin;
            if (lay_on && ye2 > 0.0f) {
                const int row = (lz * d.ncx + cxx) * d.ncy;
                if (ally) {
                    R.jb1 = start[row];
                    R.len1 = start[row + d.ncy] - R.jb1;
                } else {
                    const float ye = __builtin_amdgcn_sqrtf(ye2) + rmarg;
                    int cylo = cy + (int)floorf((yrel - ye) * inv_hyf);
                    int cyhi = cy + (int)floorf((yrel + ye) * inv_hyf);
                    cylo = max(cylo, cy - d.reach_y);
                    cyhi = min(cyhi, cy + d.reach_y);
                    const int ya = max(cylo, 0), yb = min(cyhi, d.ncy - 1);
                    if (ya <= yb) { R.jb1 = start[row + ya]; R.len1 = start[row + yb + 1] - R.jb1; }
                    if (cylo < 0) {
                        R.jb2 = start[row + cylo + d.ncy];
                        R.len2 = start[row + d.ncy] - R.jb2;
                    } else if (cyhi >= d.ncy) {
                        R.jb2 = start[row];
                        R.len2 = start[row + cyhi - d.ncy + 1] - R.jb2;
                    }
                }
            }
            R.jb1 += shift;
            R.jb2 += shift;
            return R;
        };
        // one column alone (its wrapped run too)
        auto scan_col = [&](const Runs &R) {
            scan(R.jb1, R.len1, R.jb1, 0);
            if (__ballot(R.len2 > 0) != 0) scan(R.jb2, R.len2, R.jb2, 0);
        };
        const int xlo = allx ? 0 : -d.reach, xhi = allx ? d.ncx - 1 : d.reach;
        const int ncol = xhi - xlo + 1;
        auto layer_runs = [&](int lz, int ox) {
            const float dzmin = (float)fmax(0.0, fmax(lz * d.hz - tz, tz - (lz + 1) * d.hz));
            return col_runs(lz >= lzlo && lz <= lzhi, lz, dzmin, ox);
        };
        if constexpr (SPLIT) {
            // layer by layer, this row's columns
            for (int lz = wzlo; lz <= wzhi; lz++)
                for (int ox = xlo + (int)blockIdx.y; ox <= xhi; ox += a.nsplit) scan_col(layer_runs(lz, ox));
        } else {
            for (int lz = wzlo; lz <= wzhi; lz++) {
                // columns in the order 0, -1, +1, -2, +2 (every column in
                // index order when all are searched): the first alone, then
                // pairs scanned as one sequence per lane
                auto col = [&](int i) { return allx ? i : (i == 0 ? 0 : ((i & 1) ? -((i + 1) >> 1) : (i >> 1))); };
                scan_col(layer_runs(lz, col(0)));
                for (int i = 1; i < ncol; i += 2) {
                    const Runs A = layer_runs(lz, col(i));
                    if (i + 1 < ncol) {
                        const Runs B = layer_runs(lz, col(i + 1));
                        scan(A.jb1, A.len1, B.jb1, B.len1);
                        if (__ballot(A.len2 > 0) != 0) scan(A.jb2, A.len2, A.jb2, 0);
                        if (__ballot(B.len2 > 0) != 0) scan(B.jb2, B.len2, B.jb2, 0);
                    } else {
                        scan_col(A);
                    }
                }
            }
        }
        qu.flush();
    }
    const int split = (int)(blockIdx.y + blockIdx.z * gridDim.y);
    const double fx = qu.fx, fy = qu.fy, fz = qu.fz, phi = qu.phi, dpt = qu.dpt, dpb = qu.dpb;
    double qphi = 0.0, qdt = 0.0, qdb = 0.0;
    if (active) {
        const int i = a.sidx[t];
        const double qi = me.w * d.pref;
        const double4 fo = make_double4(qi * fx, qi * fy, qi * fz, d.pref * phi);
        if (SPLIT) {
            const int64_t o = (int64_t)split * a.split_stride + i;
            a.freal_s[o] = fo;
        } else {
            a.freal[i] = fo;
        }
        qphi = qi * phi;
        if (WANT_DG) {
            qdt = qi * dpt;
            qdb = qi * dpb;
        }
    }
    // per-wave partial sums (a wave never straddles two systems)
    qphi = wave_sum(qphi);
    if (WANT_DG) { qdt = wave_sum(qdt); qdb = wave_sum(qdb); }
    if ((tid & (kWave - 1)) == 0 && t / kWave < a.n_waves) {
        const int wv = t / kWave;
        double *o = SPLIT ? a.rpart_s + 3 * ((int64_t)split * a.rsplit_stride + wv) : a.rpart + 3 * wv;
        o[0] = qphi;
        o[1] = qdt;
        o[2] = qdb;
    }
}

template <SfKind SF>
static hipError_t build_cells(rbe2d_ctx *h, const double *pos, const double *q, hipStream_t s) {
    CellArgs c;
    c.pos = pos; c.q = q; c.sys = h->w.sys; c.lay = h->w.lay; c.n_sys = h->n_sys;
    c.n_total = (int)h->n_total; c.ncells = h->total_cells;
    c.cell = h->w.cell; c.slot = h->w.slot; c.count = h->w.count; c.start = h->w.start;
    c.tmp = h->w.tmp; c.n_waves = h->n_swaves; c.sidx = h->w.sidx; c.scell = h->w.scell; c.sorted = h->w.sorted;
    // counted by the MD pass: its k-space records of these positions precede this build on s
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    c.src16 = fp32 ? h->w.src16 : nullptr;
    const bool records = h->cells_counted && h->records_moved;
    c.p32 = records && fp32 ? h->w.p32 : nullptr;
    c.p64 = records && !fp32 ? h->w.p64 : nullptr;
    const int nb = (int)((h->n_total + kBlock - 1) / kBlock);
    h->short_part = false;
    prof_begin(h, 3, s);
    // the counts start at zero (the previous build cleared them); the particle
    // pass may have counted already
    if (!h->cells_counted) hipLaunchKernelGGL(k_cell_count, dim3(nb), dim3(kBlock), 0, s, c);
    h->cells_counted = true;   // (until all launches of the build are given)
    auto built = [&] {
        const hipError_t e = hipGetLastError();
        h->cells_counted = e != hipSuccess;
        return e;
    };
    const SfArgs sf = sf_args(h);
    const int n_sf = SF == kNoSf ? 0 : SfRide<SF>::parts(sf);
    const size_t lds = (h->max_cells + 1 + (size_t)h->max_n) * sizeof(int);
    const bool many = h->n_sys > kManySystems;
    if (h->max_n <= kSmallN && lds <= kSmallLds && !(SF == kNoSf && h->n_sys >= kTinySystems && h->max_n <= kTinyN)) {
        const int threads = many && h->max_n <= kNarrowN ? kBlock : kSmallThreads, per = threads / kBlock;
        hipLaunchKernelGGL(k_cells_small<SF>, dim3(h->n_sys + (n_sf + per - 1) / per), dim3(threads),
                           std::max<size_t>(lds, per * SfRide<SF>::kLds), s, c, sf);
        prof_end(h, 3, s);
        return built();
    }
    const int nsb = (h->total_cells + kScanCells - 1) / kScanCells;
    const bool totals = nsb > kScanDirect;
    if (totals)
        hipLaunchKernelGGL(k_scan_totals, dim3(nsb), dim3(kBlock), 0, s, h->w.count, h->total_cells, h->w.scanbuf);
    hipLaunchKernelGGL(k_scan_apply, dim3(nsb), dim3(kBlock), 0, s, h->w.count, h->total_cells,
                       totals ? h->w.scanbuf : nullptr, h->w.start);
    hipLaunchKernelGGL(k_cell_scatter, dim3(nb), dim3(kBlock), 0, s, c);
    hipLaunchKernelGGL(k_cell_rank<SF>, dim3(n_sf + (h->n_swaves * kWave + kBlock - 1) / kBlock), dim3(kBlock), 0, s, c,
                       sf, n_sf);
    prof_end(h, 3, s);
    return built();
}

hipError_t launch_cells(rbe2d_ctx *h, const double *pos, const double *q, hipStream_t s) {
    return h->n_total > 0 ? build_cells<kNoSf>(h, pos, q, s) : hipSuccess;
}

// The pair sums; returns whether the assembly rode along
static bool launch_pairs(rbe2d_ctx *h, bool want_dg, const AssembleArgs *as, hipStream_t s) {
    if (h->precision != RBE2D_PREC_FP32_PHASE) {
        launch_tile_pairs(h, want_dg, as, s);
        return as != nullptr;
    }
    RealArgs r;
    r.src = h->w.sorted; r.src16 = h->w.src16; r.sidx = h->w.sidx; r.scell = h->w.scell; r.start = h->w.start;
    r.sys = h->w.sys; r.fam = h->w.fam; r.lay = h->w.lay; r.n_sys = h->n_sys; r.n_waves = h->n_swaves;
    r.freal = h->w.freal; r.rpart = h->w.rpart;
    r.freal_s = h->w.freal_s; r.rpart_s = h->w.rpart_s;
    r.split_stride = h->n_total;
    r.rsplit_stride = (int)(h->cap_sorted / kWave);
    // too few targets to fill the chip: split each target's x-columns over
    // several blocks (about 4096 waves in flight is enough)
    r.nsplit = 1;
    if (h->n_total <= h->split_cap) {
        if (h->force_rsplit) r.nsplit = h->force_rsplit;
        else if (h->tuned_now && h->tune.rsplit) r.nsplit = h->tune.rsplit;
        else r.nsplit = (int)std::min<int64_t>(kMaxRealSplit, std::max<int64_t>(1, 4096 / std::max(1, h->n_swaves)));
        r.nsplit = std::max(1, std::min(kMaxRealSplit, r.nsplit));
    }
    const int nbs = (h->n_swaves * kWave + kBlock - 1) / kBlock;
    r.nblocks = nbs;
    const int nch = 8 * RBE2D_REAL_CHUNKS;
    r.nbx = (nbs + nch - 1) / nch * nch;
    // few targets: the image families in two more layers of blocks
    int nfam = 0;
    for (const SysHost &sh : h->sys) nfam = std::max(nfam, sh.d.nfam);
    const int split = r.nsplit == 1 ? 0 : h->n_total > kFamilySplitMax ? 1 : 2;
    const int layers = split == 2 ? std::min(kMaxFamilySplit, 1 + nfam) : 1;
    h->real_parts = r.nsplit * layers;
    h->real_stride = r.rsplit_stride;
    const bool ride = as && split == 2;
    const AssembleArgs asm_args = ride ? *as : AssembleArgs();
    const int rows = r.nsplit * layers, per_row = rows * (kBlock / kWave);
    const dim3 grid(r.nbx + (ride ? (as->items() + per_row - 1) / per_row : 0), r.nsplit, layers);
    prof_begin(h, 4, s);
#define RBE2D_REAL(DG, ISO_, S, A) \
    if (want_dg == DG && h->iso == ISO_ && split == S && ride == A) \
        hipLaunchKernelGGL((k_real<DG, ISO_, S, A>), grid, dim3(kBlock), 0, s, r, asm_args);
#define RBE2D_REAL_FORMS(S, A) \
    RBE2D_REAL(false, false, S, A) RBE2D_REAL(true, false, S, A) RBE2D_REAL(false, true, S, A) RBE2D_REAL(true, true, S, A)
    RBE2D_REAL_FORMS(0, false) RBE2D_REAL_FORMS(1, false) RBE2D_REAL_FORMS(2, false) RBE2D_REAL_FORMS(2, true)
#undef RBE2D_REAL_FORMS
#undef RBE2D_REAL
    prof_end(h, 4, s);
    return ride;
}

hipError_t launch_real(rbe2d_ctx *h, const double *pos, const double *q, bool want_dg, hipStream_t s,
                       bool ride, hipEvent_t after_cells) {
    if (h->n_total == 0) return hipSuccess;
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    hipError_t e = !ride ? build_cells<kNoSf>(h, pos, q, s)
                         : fp32 ? build_cells<kSf32>(h, pos, q, s) : build_cells<kSf64>(h, pos, q, s);
    if (e == hipSuccess && after_cells) e = hipEventRecord(after_cells, s);
    if (e != hipSuccess) return e;
    if (ride) {
        const AssembleArgs as = assemble_args(h, true, nullptr);
        if (!launch_pairs(h, want_dg, &as, s)) e = launch_assemble(h, as, want_dg, s);
    } else {
        launch_pairs(h, want_dg, nullptr, s);
    }
    return e == hipSuccess ? hipGetLastError() : e;
}

// F += F_real (the pair kernel's per-particle output), and in MD steps the
// closing half kick v += dt/2 F with the completed force
// (blocks from n_blocks on: the systems' energies)
__global__ __launch_bounds__(kBlock) void k_add_real(int64_t n, RealParts real, double *F, double *vel,
                                                     double half_dt, int n_blocks, EnergyArgs en) {
    __shared__ double sh[kBlock / kWave];
    if ((int)blockIdx.x >= n_blocks) {
        energy_block(en, blockIdx.x - n_blocks, sh);
        return;
    }
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g >= n) return;
    const double4 fr = real.sum(g);
    const double add[3] = {fr.x, fr.y, fr.z};
    for (int c = 0; c < 3; c++) {
        const double f = F[3 * g + c] + add[c];
        F[3 * g + c] = f;
        if (vel) vel[3 * g + c] = fma(half_dt, f, vel[3 * g + c]);
    }
}

hipError_t launch_add_real(rbe2d_ctx *h, double *F, double *vel, double half_dt, hipStream_t s, double *energy,
                           uint32_t energy_flags) {
    if (h->n_total == 0) return hipSuccess;
    const bool ride = energy && !timed(h, 6);
    prof_begin(h, 10, s);
    const int nb = (int)((h->n_total + kBlock - 1) / kBlock);
    hipLaunchKernelGGL(k_add_real, dim3(nb + (ride ? h->n_sys : 0)), dim3(kBlock), 0, s, h->n_total, real_parts(h), F,
                       vel, half_dt, nb, energy_args(h, energy, energy_flags, nullptr, nullptr));
    prof_end(h, 10, s);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess && energy && !ride ? launch_energy(h, energy, energy_flags, nullptr, nullptr, s) : e;
}

}  // namespace rbe2d
