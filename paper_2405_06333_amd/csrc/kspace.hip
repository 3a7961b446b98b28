// k-space half of RBE2D on gfx950: particle preparation, the N x P
// structure-factor pass, the FP64 reduction/recalibration per k, the force
// scatter.  Every launch covers all systems of a handle; a block finds its
// system in the layout tables (particles are padded per system to whole
// tiles, so blocks never straddle systems and k-data stay wave-uniform).
//
// Phases are carried in revolutions: k.r / 2pi = nx fx + ny fy + nz fz with
// fx = x/Lx wrapped into [0,1), fy = y/Ly, fz = z/Lz_ext.
//  * FP32 path: f is split into fh (fh_bits = 22 - b fraction bits, where
//    every |n| < 2^b) and fl = f - fh.  Then n fh has at most 22 significant
//    bits and nx fxh + ny fyh at most 23, so both are exact in FP32; the
//    phase fract(nx fxh + ny fyh) + nx fxl + ny fyl (and likewise in z)
//    keeps ~1e-8 revolution accuracy, and the hardware v_sin_f32/v_cos_f32
//    take revolutions directly.
//  * FP64 path: plain FP64 phases, sine and cosine from devmath.h.
#include <algorithm>
#include <type_traits>

#include "devmath.h"
#include "energy.h"
#include "kspace_dev.h"
#include "rbe2d_internal.h"
#include "sampler.h"

namespace rbe2d {

// ---------------------------------------------------------------------------
// k-vector tables (nx, ny, nz as floats / doubles, padded with zeros), of the
// k-set at hand or of one drawn here
// ---------------------------------------------------------------------------

struct TableArgs {
    SampleArgs sample;       // the k-set, and how to draw it when `draw` is set
    int draw, P_pad, chunk, chunks;
    float4 *kn32;
    double4 *kn64;
};

__device__ __forceinline__ int3 table_kvec(const TableArgs &a, int r, int l) {
    int32_t *k = a.sample.kset + 3 * ((int64_t)r * a.sample.P + l);
    if (!a.draw) return make_int3(k[0], k[1], k[2]);
    const int3 n = draw_kvec(a.sample, r, l);
    k[0] = n.x; k[1] = n.y; k[2] = n.z;
    return n;
}

// FP32: kBlock entries of the systems' tables
__device__ __forceinline__ void table32(const TableArgs &a, int blk) {
    const int kg = blk * kBlock + threadIdx.x;
    if (kg >= a.sample.n_sys * a.P_pad) return;
    const int r = kg / a.P_pad, l = kg - r * a.P_pad;
    int3 n = make_int3(0, 0, 0);
    if (l < a.sample.P) n = table_kvec(a, r, l);
    a.kn32[kg] = make_float4((float)n.x, (float)n.y, (float)n.z, 0.0f);
}

// FP64: the k-vectors of system r sorted by |nz| in chunks (z_chunk), (nx, ny,
// |nz|, +-(1 + index in the k-set) with the sign of nz), by a counting sort in
// LDS, one block per chunk.  |nz| beyond the last bucket are left unsorted: the
// structure-factor pass compares neighbours and only saves less, as it does at
// the ends of a chunk.  (The order within a bucket is that of the LDS atomics;
// no sum depends on it.)
constexpr int kZBuckets = 2048;
__device__ __forceinline__ int z_bucket(int nz) { return min(abs(nz), kZBuckets - 1); }
__device__ void table64(const TableArgs &a, int blk) {
    __shared__ int count[kZBuckets];
    __shared__ int sh[kBlock / 64];
    const int r = a.chunks == 1 ? blk : blk / a.chunks, l0 = (blk - r * a.chunks) * a.chunk;
    const int l1 = min(a.sample.P, l0 + a.chunk), pad1 = min(a.P_pad, l0 + a.chunk);
    const int32_t *k = a.sample.kset + 3 * (int64_t)r * a.sample.P;
    constexpr int kPer = kZBuckets / kBlock;
#pragma unroll
    for (int b = 0; b < kPer; b++) count[b * kBlock + threadIdx.x] = 0;
    __syncthreads();
    for (int l = l0 + threadIdx.x; l < l1; l += kBlock) atomicAdd(&count[z_bucket(table_kvec(a, r, l).z)], 1);
    __syncthreads();
    int v[kPer], t = 0;
#pragma unroll
    for (int b = 0; b < kPer; b++) { v[b] = count[kPer * threadIdx.x + b]; t += v[b]; }
    int run = block_scan(t, sh);
#pragma unroll
    for (int b = 0; b < kPer; b++) { count[kPer * threadIdx.x + b] = run; run += v[b]; }
    __syncthreads();
    double4 *o = a.kn64 + (int64_t)r * a.P_pad;
    for (int l = l0 + threadIdx.x; l < pad1; l += kBlock) {
        if (l < l1) {
            // (a drawn k-vector was written by this thread)
            const int nx = k[3 * l], ny = k[3 * l + 1], nz = k[3 * l + 2];
            const int at = l0 + atomicAdd(&count[z_bucket(nz)], 1);
            o[at] = make_double4((double)nx, (double)ny, fabs((double)nz), nz < 0 ? -1.0 - l : 1.0 + l);
        } else {
            o[l] = make_double4(0.0, 0.0, 0.0, 0.0);
        }
    }
}

// ---------------------------------------------------------------------------
// 1. particle preparation
// ---------------------------------------------------------------------------

struct PrepArgs {
    const double *pos, *q;
    const SysDesc *sys;
    Layout lay;
    int n_sys;
    float4 *p32;
    double4 *p64;
    double *bpart;
    int *err;
    // MD update first (MD > 0): positions and velocities are updated in place
    double *pos_md, *vel;
    const double *F;
    RealParts real;             // MD == 2: the pair kernel's part of the force
    double dt, zlo, zhi_from_top;
    // with count set: the cell and in-cell slot of each (moved) particle for
    // the next cell-list build (the counts start at zero)
    int *cell, *slot, *count;
    // MD == 3: the Langevin update's parameters
    double c1, c2;
    uint64_t seed, stream_base;
    const long long *dev_step;
    int n_tblocks;              // the first blocks write the k-vector tables (one draw is a long chain)
    TableArgs tab;
};

// r += dt/2 v; v = c1 v + c2 xi; r += dt/2 v; wrap / reflect, after the kick
// v += dt/2 F (Langevin equation, unit masses).  xi: Box-Muller normals from
// the SplitMix64 stream (seed, 2^63 + step n_sys + system), uniforms 2(3i+c)
// and 2(3i+c)+1 for particle i of its system.
__device__ __forceinline__ void langevin_drift(const SysDesc &d, const PrepArgs &a, int r, int local, double (&v)[3],
                                               double (&x)[3]) {
    const uint64_t base = a.dev_step ? (uint64_t)(*a.dev_step) * (uint64_t)a.n_sys : a.stream_base;
    const uint64_t key = stream_key(a.seed, kThermoStream + base + (uint64_t)r);
    const double h = 0.5 * a.dt;
    for (int c = 0; c < 3; c++) {
        x[c] = fma(h, v[c], x[c]);
        const uint64_t k = 3 * (uint64_t)local + c;
        const double u1 = uniform01(key, 2 * k), u2 = uniform01(key, 2 * k + 1);
        const double xi = sqrt(-2.0 * log(1.0 - u1)) * cos(2.0 * kPi * u2);
        v[c] = fma(a.c1, v[c], a.c2 * xi);
        x[c] = fma(h, v[c], x[c]);
    }
    x[0] -= d.Lx * floor(x[0] / d.Lx);
    x[1] -= d.Ly * floor(x[1] / d.Ly);
    const double zlo = a.zlo, zhi = d.H - a.zhi_from_top;
    const double W = zhi - zlo;
    const double u = x[2] - zlo;
    const double m = floor(u / W);
    const double rem = u - m * W;
    const bool odd = fmod(fabs(m), 2.0) == 1.0;
    x[2] = odd ? zhi - rem : zlo + rem;
    if (odd) v[2] = -v[2];
    x[2] = fmin(fmax(x[2], zlo), zhi);
}

// MD: 0 none; 1 opening half kick with F and drift; 2 closing half kick and
// the next opening half kick, both with F + freal (the same force, the same
// roundings as two separate kicks), and drift; 3 the Langevin update up to the
// force evaluation (BAOAB).  Then the k-space particle records of the (new)
// positions, their cells and the block sums of the IBC.  The k-vector tables,
// and with an MD update the draw of the k-set, are blocks of the same launch:
// a call of a few thousand particles lasts about as long as its launches take
// to issue (6 to 7 us each).
template <bool FP32, int MD>
__global__ __launch_bounds__(kBlock) void k_prep(PrepArgs a) {
    __shared__ double sh[4][kBlock / 64];
    if ((int)blockIdx.x < a.n_tblocks) {
        if (FP32) table32(a.tab, blockIdx.x);
        else table64(a.tab, blockIdx.x);
        return;
    }
    const int b = blockIdx.x - a.n_tblocks;
    const int r = find_sys(a.lay.bbase, a.n_sys, b);
    const SysDesc &d = a.sys[r];
    const int iloc = (b - a.lay.bbase[r]) * kBlock + threadIdx.x;
    const int Nr = a.lay.off[r + 1] - a.lay.off[r];
    const int64_t ii = (int64_t)a.lay.pbase[r] + iloc;      // internal (padded) index
    double sqz = 0.0, sq = 0.0, sq2 = 0.0, sqzz = 0.0;
    double fx = 0, fy = 0, fz = 0, qi = 0;
    if (iloc < Nr) {
        const int64_t g = (int64_t)a.lay.off[r] + iloc;      // caller index
        double x, y, z;
        if (MD > 0) {
            double v[3], rr[3], add[3] = {0.0, 0.0, 0.0};
            if (MD == 2) {
                const double4 fr = a.real.sum(g);
                add[0] = fr.x; add[1] = fr.y; add[2] = fr.z;
            }
            for (int c = 0; c < 3; c++) {
                const double f = MD == 2 ? a.F[3 * g + c] + add[c] : a.F[3 * g + c];
                v[c] = fma(0.5 * a.dt, f, a.vel[3 * g + c]);
                if (MD == 2) v[c] = fma(0.5 * a.dt, f, v[c]);
                rr[c] = a.pos_md[3 * g + c];
            }
            if (MD == 3) langevin_drift(d, a, r, iloc, v, rr);
            else drift_fold(d, a.dt, a.zlo, a.zhi_from_top, v, rr);
            for (int c = 0; c < 3; c++) {
                a.vel[3 * g + c] = v[c];
                a.pos_md[3 * g + c] = rr[c];
            }
            x = rr[0]; y = rr[1]; z = rr[2];
        } else {
            x = a.pos[3 * g]; y = a.pos[3 * g + 1]; z = a.pos[3 * g + 2];
        }
        if (a.count) {
            const int c = d.cbase + cell_of(x, y, z, d);
            a.cell[g] = c;
            a.slot[g] = atomicAdd(&a.count[c], 1);
        }
        qi = a.q[g];
        if (!(z > 0.0 && z < d.H)) atomicOr(a.err, 1);
        fx = x * d.inv_Lx; fx -= floor(fx);
        fy = y * d.inv_Ly; fy -= floor(fy);
        fz = z * d.inv_Lz;
        sqz = qi * z; sq = qi; sq2 = qi * qi; sqzz = qi * z * z;
    }
    if (FP32) {
        // scale_h = 2^fh_bits: the split is exact
        const double hx = ldexp(rint(fx * d.scale_h), -d.fh_bits);
        const double hy = ldexp(rint(fy * d.scale_h), -d.fh_bits);
        const double hz = ldexp(rint(fz * d.scale_h), -d.fh_bits);
        a.p32[2 * ii] = make_float4((float)hx, (float)(fx - hx), (float)hy, (float)(fy - hy));
        a.p32[2 * ii + 1] = make_float4((float)hz, (float)(fz - hz), (float)qi, 0.0f);
    } else {
        a.p64[ii] = make_double4(fx, fy, fz, qi);
    }
    // block sums of q z, q, q^2, q z^2 (one barrier for the four)
    sqz = wave_sum(sqz);
    sq = wave_sum(sq);
    sq2 = wave_sum(sq2);
    sqzz = wave_sum(sqzz);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) { sh[0][wid] = sqz; sh[1][wid] = sq; sh[2][wid] = sq2; sh[3][wid] = sqzz; }
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int k = 0; k < kBlock / 64; k++) t += sh[threadIdx.x][k];
        a.bpart[4 * b + threadIdx.x] = t;
    }
}

__global__ __launch_bounds__(64) void k_scalars(ScalArgs a) { ibc_scalars(a, blockIdx.x, threadIdx.x); }

// Wave vectors per block of the FP64 table.  One block for all of a system is a
// chain that every other launch waits for, 11 us per 256 draws; every block more
// takes sines from the structure-factor pass (sorted by 512 instead of 1024: 2
// to 3 % of it).  Velocity-Verlet steps by all | 1024 | 512: 500 ions, P = 4096
// 142 | 110 | 104 us, P = 1000 88 | 88 | 82, 4000 ions, P = 16000 611 | 333 |
// 331, 40000 ions, P = 1000 193 | 193 | 188, 300000 ions 944 | 945 | 958.
static int z_chunk(const rbe2d_ctx *h, bool draw) { return draw && h->n_total <= 100000 ? 512 : 1024; }

static PrepArgs prep_args(rbe2d_ctx *h, const double *pos, const double *q, bool draw) {
    PrepArgs a{};
    a.pos = pos; a.q = q; a.sys = h->w.sys; a.lay = h->w.lay; a.n_sys = h->n_sys;
    a.p32 = h->w.p32; a.p64 = h->w.p64; a.bpart = h->w.bpart; a.err = h->w.err;
    a.cell = h->w.cell; a.slot = h->w.slot;
    a.tab.sample = sample_args(h, 0, 0, nullptr);
    a.tab.P_pad = h->P_pad; a.tab.kn32 = h->w.kn32; a.tab.kn64 = h->w.kn64;
    a.tab.draw = draw; a.tab.chunk = z_chunk(h, draw); a.tab.chunks = (h->P_pad + a.tab.chunk - 1) / a.tab.chunk;
    // (the call without a handle may go without a k-set, and then without k-space)
    if (h->w.kset)
        a.n_tblocks = h->precision == RBE2D_PREC_FP32_PHASE ? (h->n_sys * h->P_pad + kBlock - 1) / kBlock
                                                            : h->n_sys * a.tab.chunks;
    return a;
}

ScalArgs scal_args(rbe2d_ctx *h) {
    ScalArgs b;
    b.bpart = h->w.bpart; b.sys = h->w.sys; b.lay = h->w.lay; b.scal = h->w.scal;
    return b;
}

static void launch_scalars(rbe2d_ctx *h, hipStream_t s) {
    hipLaunchKernelGGL(k_scalars, dim3(h->n_sys), dim3(64), 0, s, scal_args(h));
}

template <int MD>
static void launch_prep_kernel(rbe2d_ctx *h, const PrepArgs &a, hipStream_t s) {
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    const dim3 g(a.n_tblocks + h->n_blocks);
    if (g.x == 0) return;
    if (fp32) hipLaunchKernelGGL((k_prep<true, MD>), g, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_prep<false, MD>), g, dim3(kBlock), 0, s, a);
}

hipError_t launch_prep(rbe2d_ctx *h, const double *pos, const double *q, hipStream_t s, bool scalars, bool count) {
    prof_begin(h, 0, s);
    PrepArgs a = prep_args(h, pos, q, false);
    if (count) a.count = h->w.count;
    launch_prep_kernel<0>(h, a, s);
    if (count) {
        h->cells_counted = h->n_total > 0;
        h->records_moved = false;
    }
    if (scalars) launch_scalars(h, s);
    prof_end(h, 0, s);
    return hipGetLastError();
}

hipError_t launch_prep_md(rbe2d_ctx *h, int md, double *pos, double *vel, const double *F, const double *q, double dt,
                          double zlo, double zhi_from_top, const MdExtra *mx, uint64_t seed, uint64_t stream_base,
                          const long long *dev_step, hipStream_t s) {
    const bool draw = !timed(h, 8);
    if (!draw) {
        const hipError_t e = launch_sample(h, seed, stream_base, dev_step, s);
        if (e != hipSuccess) return e;
    }
    PrepArgs a = prep_args(h, pos, q, draw);
    a.pos_md = pos; a.vel = vel; a.F = F; a.real = real_parts(h);
    a.dt = dt; a.zlo = zlo; a.zhi_from_top = zhi_from_top;
    // a force evaluation with real space follows: count the particles per
    // cell here, where their new positions are at hand
    a.count = h->w.count;
    a.tab.sample = sample_args(h, seed, stream_base, dev_step);
    if (md == 3) {
        a.c1 = mx->c1; a.c2 = mx->c2; a.seed = seed; a.stream_base = stream_base; a.dev_step = dev_step;
    }
    prof_begin(h, 7, s);
    if (md == 1) launch_prep_kernel<1>(h, a, s);
    else if (md == 2) launch_prep_kernel<2>(h, a, s);
    else launch_prep_kernel<3>(h, a, s);
    prof_end(h, 7, s);
    h->cells_counted = h->n_total > 0;
    h->records_moved = md != 3;
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 2. structure-factor pass: per (particle tile, k-chunk) partial sums of
//    rho(k) = sum q e^{2 pi i phi} and rhohat(k) = sum q e^{2 pi i phihat}
//    with phi = phi_xy + phi_z, phihat = phi_xy - phi_z.
//    Lanes own particles, the k-chunk is wave-uniform (scalar loads).
// ---------------------------------------------------------------------------

// One block per (tile, k-chunk): kspace_dev.h.
template <int KC>
__global__ __launch_bounds__(kBlock) void k_sf32(const float4 *__restrict__ p32,
                                                 const float4 *__restrict__ kn, const int *tbase,
                                                 int n_sys, int per_thread, int P_pad, int n_tiles,
                                                 double *__restrict__ part) {
    __shared__ SfLds32<KC> lds;
    const TileChunk tc = tile_chunk((int)blockIdx.x, P_pad / KC);
    if (tc.tile >= n_tiles) return;
    sf32_block<KC, false>(p32, kn, tbase, n_sys, per_thread, P_pad, part, tc, threadIdx.x, lds.sh);
}
template <int KC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_sf64(const double4 *__restrict__ p64,
                                                 const double4 *__restrict__ ks, const int *tbase,
                                                 int n_sys, int per_thread, int P_pad, int n_tiles,
                                                 double *__restrict__ part) {
    __shared__ SfLds64<KC> lds;
    const TileChunk tc = tile_chunk((int)blockIdx.x, P_pad / KC);
    if (tc.tile >= n_tiles) return;
    sf64_block<KC, false>(p64, ks, tbase, n_sys, per_thread, P_pad, part, tc, threadIdx.x, lds.sh, lds.tab);
}

// ---------------------------------------------------------------------------
// 3. reduce over tiles (FP64, fixed order) and recalibrate (Sec. 3.4):
//    rho^M = (1 + Y_even) rho + Y_odd rhohat,
//    A = rho^M + (1 + conj Y_even) rho,  B = conj(Y_odd) rho,
//    c = 2 pi S pref / (V P |k|^2),  e = c Re(rho conj(rho^M)).
//    One wave per (system, k); lanes split the tiles and the image orders.
// ---------------------------------------------------------------------------

template <bool DG>
__global__ __launch_bounds__(64) void k_assemble(AssembleArgs a) {
    assemble_wave<DG>(a, blockIdx.x, threadIdx.x);
}

int choose_tile(int64_t N, int n_kchunks) {
    // particles per thread: fill the chip with >= ~4096 blocks if N allows,
    // but keep tiles long enough to amortise the block reduction.
    int per = kMaxTileThreads;
    while (per > 1) {
        const int64_t tiles = (N + (int64_t)kBlock * per - 1) / ((int64_t)kBlock * per);
        if (tiles * n_kchunks >= 4096) break;
        per >>= 1;
    }
    return per;
}

SfArgs sf_args(rbe2d_ctx *h) {
    SfArgs a;
    a.p32 = h->w.p32; a.p64 = h->w.p64; a.kn32 = h->w.kn32; a.kn64 = h->w.kn64; a.tbase = h->w.lay.tbase;
    a.n_sys = h->n_sys; a.per = h->per; a.P_pad = h->P_pad; a.n_tiles = h->n_tiles;
    a.part = (double *)h->w.sfpart;
    return a;
}

AssembleArgs assemble_args(rbe2d_ctx *h, bool with_scalars, long long *step) {
    AssembleArgs a;
    a.part = (const double *)h->w.sfpart; a.P = h->P; a.P_pad = h->P_pad;
    a.tbase = h->w.lay.tbase; a.kset = h->w.kset; a.sys = h->w.sys; a.img = h->w.img;
    a.krec = h->w.krec; a.kf32 = h->w.kf32;
    a.kf64 = h->precision == RBE2D_PREC_FP32_PHASE ? nullptr : h->w.kf64;
    a.n_sys = h->n_sys; a.with_scalars = with_scalars; a.sc = scal_args(h);
    a.step = step;
    return a;
}

hipError_t launch_kcoef_sf(rbe2d_ctx *h, hipStream_t s, bool with_scalars, bool want_dg, long long *step) {
    prof_begin(h, 1, s);
    if (h->n_tiles > 0) {
        const SfArgs a = sf_args(h);
        const int tiles8 = (h->n_tiles + 7) / 8 * 8;
        if (h->precision == RBE2D_PREC_FP32_PHASE)
            hipLaunchKernelGGL(k_sf32<kKChunk32>, dim3((unsigned)tiles8 * (h->P_pad / kKChunk32)), dim3(kBlock), 0, s,
                               a.p32, a.kn32, a.tbase, a.n_sys, a.per, a.P_pad, a.n_tiles, a.part);
        else
            hipLaunchKernelGGL(k_sf64<kKChunk64>, dim3((unsigned)tiles8 * (h->P_pad / kKChunk64)), dim3(kBlock), 0, s,
                               a.p64, a.kn64, a.tbase, a.n_sys, a.per, a.P_pad, a.n_tiles, a.part);
    }
    prof_end(h, 1, s);
    return launch_assemble(h, assemble_args(h, with_scalars, step), want_dg, s);
}

hipError_t launch_assemble(rbe2d_ctx *h, const AssembleArgs &a, bool want_dg, hipStream_t s) {
    prof_begin(h, 2, s);
    if (want_dg) hipLaunchKernelGGL(k_assemble<true>, dim3(a.items()), dim3(64), 0, s, a);
    else hipLaunchKernelGGL(k_assemble<false>, dim3(a.items()), dim3(64), 0, s, a);
    prof_end(h, 2, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 4. force scatter: one thread per particle, all k (or a k-range) uniform:
//    F_i = -q_i sum_l [k_l Im(e^{-i phi} cA_l) + khat_l Im(e^{-i phihat} cB_l)]
//    pot_i = sum_l [Re(e^{-i phi} cA_l) + Re(e^{-i phihat} cB_l)]   (dE_k/dq_i)
// ---------------------------------------------------------------------------

struct ForceArgs {
    const float4 *p32;
    const double4 *p64;
    const float4 *kn32;
    const float4 *kf32;
    const double *kf64;
    Layout lay;
    const SysDesc *sys;
    int n_sys, P, P_pad;
    int split, k_per_split;  // the k-range in `split` parts of k_per_split
    const double *pos;       // for the IBC potential (z_i)
    const double *q;
    const double *scal;
    RealParts real;          // added when add_real
    double *F;               // final output (caller order, N x 3)
    double *dEdq;            // final dE/dq when want_pot
    double *var;             // force-variance estimate per particle (variance mode)
    const double *gE;        // scale of the backward outputs (device scalar) or null
    int accumulate, add_real, want_pot, want_var, do_kspace, do_ibc;
    // kWaves: blocks from n_groups on form the systems' energies (k_force_rows:
    // from n_blocks on); *err goes to err_out when set
    int n_groups;
    EnergyArgs en;
    const int *err;
    int32_t *err_out;
    double4 *part;           // kRows: sums of the block rows, part_stride apart
    int64_t part_stride;
    int rows;
};

// f: the sums over k (times q_i and with the real-space part: force_terms)
__device__ __forceinline__ double4 force_terms(const ForceArgs &a, double qi, const double4 &f,
                                               const double4 &real) {
    if (a.want_var || !a.do_kspace) return a.want_var ? f : real;
    return make_double4(fma(-qi, f.x, real.x), fma(-qi, f.y, real.y), fma(-qi, f.z, real.z), real.w + f.w);
}

__device__ __forceinline__ void finish_particle(const ForceArgs &a, int r, int64_t g, double qi, const double4 &f) {
    const SysDesc &d = a.sys[r];
    const double *sc = a.scal + kScal * r;
    if (a.want_var) {
        // f.w carries sum_l |t_l|^2 / q_i^2: (P sum |t|^2 - |F|^2) / (P - 1)
        const double P = (double)a.P;
        a.var[g] = a.P > 1 ? qi * qi * (P * f.w - (f.x * f.x + f.y * f.y + f.z * f.z)) / (P - 1.0) : 0.0;
        return;
    }
    double Fx = f.x, Fy = f.y, Fz = f.z, ph = f.w;
    if (a.do_kspace) ph -= 2.0 * d.alpha * d.pref / sqrt(kPi) * qi;   // + dE_self/dq_i
    if (a.do_ibc) {
        if (d.surf) {
            // IBC with the surface terms: linear (and quadratic) in z
            const double z = a.pos[3 * g + 2];
            Fz += qi * (sc[4] + sc[10] + sc[9] * z);
            ph += -sc[4] * z + sc[5] + sc[11] + z * (sc[12] + sc[13] * z);
        } else {
            Fz += qi * sc[4];
            ph += -sc[4] * a.pos[3 * g + 2] + sc[5];
        }
    }
    if (a.want_pot) {
        // backward: dL/dr = -gE F, dL/dq = gE phi
        const double gs = a.gE ? *a.gE : 1.0;
        if (a.F) {
            a.F[3 * g] = -gs * Fx; a.F[3 * g + 1] = -gs * Fy; a.F[3 * g + 2] = -gs * Fz;
        }
        if (a.dEdq) a.dEdq[g] = gs * ph;
        return;
    }
    const double o[3] = {Fx, Fy, Fz};
    for (int c = 0; c < 3; c++) {
        a.F[3 * g + c] = a.accumulate ? a.F[3 * g + c] + o[c] : o[c];
    }
}

// Blocks of the force pass.  kWhole: one thread per particle takes all k.
// kWaves (too few particles to fill the chip): the waves of a block share 64
// particles and take the parts of the k-range in turn, and their sums meet in
// LDS: 32 KB at most, where sums kept in memory for a second launch cost that
// launch (6 us of a call of 60 to 100 us).  kRows: with many wave vectors (P
// beyond kLongP) the parts are what a call lasts, on the N / 64 CUs that hold
// those blocks; rows of blocks of 4 waves then take one part each, over the
// whole chip, and a second launch adds the rows.  K-space forces, kWaves |
// kRows: 500 ions, P = 4096 FP64 148 | 75 and FP32 79 | 44 us, 4000 ions, P =
// 2000 89 | 58 and 49 | 39, P = 1024 53 | 40 and 32 | 30, P = 600 37 | 34 and
// 25 | 27.
enum ForceSplit { kWhole, kWaves, kRows };
constexpr int kMaxForceWaves = 16, kRowWaves = 4;
template <ForceSplit SPLIT, typename Sum>
__device__ __forceinline__ void force_block(const ForceArgs &a, Sum sum) {
    extern __shared__ __align__(16) double fsh[];
    if constexpr (SPLIT != kWhole) {
        if (SPLIT == kWaves && (int)blockIdx.x >= a.n_groups) {
            energy_block(a.en, blockIdx.x - a.n_groups, fsh);
            return;
        }
        const int lane = threadIdx.x & (kWave - 1);
        const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (the k-records come by scalar loads)
        const int b = blockIdx.x / (kBlock / kWave);
        const int r = find_sys(a.lay.bbase, a.n_sys, b);
        const int first = (b - a.lay.bbase[r]) * kBlock + (blockIdx.x % (kBlock / kWave)) * kWave;
        const int Nr = a.lay.off[r + 1] - a.lay.off[r];
        if (first >= Nr) return;
        const int64_t ii = (int64_t)a.lay.pbase[r] + first + lane;   // (the records are padded)
        const bool on = first + lane < Nr;
        const int64_t g = (int64_t)a.lay.off[r] + first + (on ? lane : 0);
        const int nw = blockDim.x / kWave;
        const double qi = a.q[g];
        // the parts of the real-space forces too are dealt to the waves
        double4 real = make_double4(0.0, 0.0, 0.0, 0.0), f = real;
        if (SPLIT == kWaves && a.add_real)
            for (int p = wid; p < a.real.n; p += nw) {
                const double4 v = a.real.f[p * a.real.stride + g];
                real.x += v.x; real.y += v.y; real.z += v.z; real.w += v.w;
            }
        if (SPLIT == kWaves && a.add_real && a.real.more && wid == 0) {
            const double4 v = a.real.more[g];
            real.x += v.x; real.y += v.y; real.z += v.z;
        }
        if (a.do_kspace)
            for (int k = wid + (SPLIT == kRows ? (int)blockIdx.y * nw : 0); k < a.split; k += SPLIT == kRows ? a.rows * nw : nw)
                sum(r, ii, k * a.k_per_split, min(a.P, (k + 1) * a.k_per_split), f);
        // (stores only from here on: the loads above stay scalar)
        if (SPLIT == kWaves && a.err_out && blockIdx.x == 0 && threadIdx.x == 0) *a.err_out = *a.err;
        double4 *part = reinterpret_cast<double4 *>(fsh);
        if (SPLIT == kWaves) f = force_terms(a, qi, f, real);
        part[threadIdx.x] = f;
        __syncthreads();
        if (wid != 0 || !on) return;
        for (int w = 1; w < nw; w++) {
            const double4 v = part[w * kWave + lane];
            f.x += v.x; f.y += v.y; f.z += v.z; f.w += v.w;
        }
        if (SPLIT == kRows) a.part[blockIdx.y * a.part_stride + ii] = f;
        else finish_particle(a, r, g, qi, f);
    } else {
        const int b = blockIdx.x;
        const int r = find_sys(a.lay.bbase, a.n_sys, b);
        const int iloc = (b - a.lay.bbase[r]) * kBlock + threadIdx.x;
        if (iloc >= a.lay.off[r + 1] - a.lay.off[r]) return;
        double4 f = make_double4(0.0, 0.0, 0.0, 0.0);
        if (a.do_kspace) sum(r, (int64_t)a.lay.pbase[r] + iloc, 0, a.P, f);
        const int64_t g = (int64_t)a.lay.off[r] + iloc;
        const double qi = a.q[g];
        finish_particle(a, r, g, qi, force_terms(a, qi, f, a.add_real ? a.real.sum<1>(g) : make_double4(0, 0, 0, 0)));
    }
}

// The rows' sums of a force pass in rows, in their order, and what ends the pass
__global__ __launch_bounds__(kBlock) void k_force_rows(ForceArgs a, int n_blocks) {
    __shared__ double sh[kBlock / kWave];
    if ((int)blockIdx.x >= n_blocks) {
        energy_block(a.en, blockIdx.x - n_blocks, sh);
        return;
    }
    const int b = blockIdx.x;
    const int r = find_sys(a.lay.bbase, a.n_sys, b);
    const int iloc = (b - a.lay.bbase[r]) * kBlock + threadIdx.x;
    if (iloc >= a.lay.off[r + 1] - a.lay.off[r]) return;
    const double4 *p = a.part + a.lay.pbase[r] + iloc;
    double4 f = p[0];
    for (int y = 1; y < a.rows; y++) {
        const double4 v = p[y * a.part_stride];
        f.x += v.x; f.y += v.y; f.z += v.z; f.w += v.w;
    }
    const int64_t g = (int64_t)a.lay.off[r] + iloc;
    const double qi = a.q[g];
    finish_particle(a, r, g, qi, force_terms(a, qi, f, a.add_real ? a.real.sum(g) : make_double4(0, 0, 0, 0)));
}

// MODE 0: forces; 1: forces and potentials (adjoint); 2: forces and the sum
// of the squared per-k force terms (variance estimate)
template <int MODE, ForceSplit SPLIT>
__global__ __launch_bounds__(SPLIT == kWaves ? kMaxForceWaves * kWave : kBlock) void k_force32(ForceArgs a) {
    force_block<SPLIT>(a, [&](int r, int64_t ii, int l0, int l1, double4 &F) {
        const float4 pa = a.p32[2 * ii];
        const float4 pb = a.p32[2 * ii + 1];
        const float4 *kn = a.kn32 + (int64_t)r * a.P_pad;
        const float4 *kf = a.kf32 + 3 * (int64_t)r * a.P;
        // per k: n (kn), k and |k_xy|^2 (kv), and the amplitudes (ab for the
        // potentials, else their polar form)
        constexpr int kExtra = MODE == 1 ? 1 : 2;
        float fx = 0, fy = 0, fz = 0, pt = 0;
        auto one = [&](const float4 &n, const float4 &kv, const float4 &ex) {
            float pxy = fractf(fmaf(n.y, pa.z, n.x * pa.x));
            pxy = fmaf(n.x, pa.y, pxy);
            pxy = fmaf(n.y, pa.w, pxy);
            const float pz = fmaf(n.z, pb.y, fractf(n.z * pb.x));
            float X, Y;   // Im(e^{-i ph} cA), Im(e^{-i phh} cB)
            if (MODE == 1) {
                // the potential needs the real parts too (ex = cA, cB)
                const float ph = pxy + pz, phh = pxy - pz;
                const float c1f = cos_rev(ph), s1f = sin_rev(ph);
                const float c2f = cos_rev(phh), s2f = sin_rev(phh);
                X = fmaf(ex.y, c1f, -ex.x * s1f);
                Y = fmaf(ex.w, c2f, -ex.z * s2f);
                pt = fmaf(ex.x, c1f, pt); pt = fmaf(ex.y, s1f, pt);
                pt = fmaf(ex.z, c2f, pt); pt = fmaf(ex.w, s2f, pt);
            } else {
                // polar form: one transcendental per product
                X = ex.x * sin_rev((ex.y - pxy) - pz);
                Y = ex.z * sin_rev((ex.w - pxy) + pz);
            }
            const float sp = X + Y, sm = X - Y;
            fx = fmaf(kv.x, sp, fx);
            fy = fmaf(kv.y, sp, fy);
            fz = fmaf(kv.z, sm, fz);
            if (MODE == 2) pt = fmaf(kv.w * sp, sp, fmaf(kv.z * sm, kv.z * sm, pt));
        };
        for (int c0 = l0; c0 < l1; c0 += 64) {
            const int c1 = min(l1, c0 + 64);
            fx = fy = fz = pt = 0;
            int l = c0;
            // four k at a time: their records are fetched together (scalar
            // loads), one wait per four instead of one per k
            for (; l + 4 <= c1; l += 4) {
                float4 n[4], kv[4], ex[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    n[j] = record(kn + l + j);
                    kv[j] = record(kf + 3 * (l + j));
                    ex[j] = record(kf + 3 * (l + j) + kExtra);
                }
#pragma unroll
                for (int j = 0; j < 4; j++) one(n[j], kv[j], ex[j]);
            }
            for (; l < c1; l++) one(record(kn + l), record(kf + 3 * l), record(kf + 3 * l + kExtra));
            F.x += fx; F.y += fy; F.z += fz; F.w += pt;
        }
    });
}

// FP64.  The wave vectors enter as integers, n = (nx, ny, nz), and the sums are
// scaled by 2 pi / L at the end: one 64-byte record per k (MODE 1: and 32 bytes
// of amplitudes) comes by scalar loads, where k, n and the amplitudes of the
// per-k records took 112 bytes from two arrays.  Bound by VALU issue, 40
// instructions per (particle, k), two sines; 1e6 ions, P = 500: 0.61 ms
// instead of 0.72 (46 instructions).
template <int MODE, ForceSplit SPLIT>
__global__ __launch_bounds__(SPLIT == kWaves ? kMaxForceWaves * kWave : kBlock) void k_force64(ForceArgs a) {
    using Record = std::conditional_t<SPLIT != kWhole, ConstDouble, double>;
    __shared__ double2 tab[MODE == 1 ? kParts : 1];
    if (MODE == 1) {
        if (threadIdx.x < kParts)
            tab[threadIdx.x] = make_double2(kPartTable[threadIdx.x][0], kPartTable[threadIdx.x][1]);
        __syncthreads();
    }
    force_block<SPLIT>(a, [&](int r, int64_t ii, int l0, int l1, double4 &F) {
        const double4 p = a.p64[ii];
        const double *kf = a.kf64 + (int64_t)r * a.P * kKF64;
        const SysDesc &d = a.sys[r];
        const double wx = 2.0 * kPi * d.inv_Lx, wy = 2.0 * kPi * d.inv_Ly, wz = 2.0 * kPi * d.inv_Lz;
        double fx = 0, fy = 0, fz = 0, pt = 0;
        for (int l = l0; l < l1; l++) {
            const Record *f = (const Record *)(kf + (int64_t)l * kKF64);
            const double nx = f[0], ny = f[1], nz = f[2];
            const double pxy = fma(ny, p.y, nx * p.x);
            double X, Y;   // Im(e^{-i ph} cA), Im(e^{-i phh} cB)
            if (MODE == 1) {
                // the potential needs the real parts too
                double c1, s1, c2, s2;
                sincos_table64(fma(nz, p.z, pxy), tab, &s1, &c1);
                sincos_table64(fma(-nz, p.z, pxy), tab, &s2, &c2);
                X = fma(f[9], c1, -f[8] * s1);
                Y = fma(f[11], c2, -f[10] * s2);
                pt = fma(f[8], c1, pt); pt = fma(f[9], s1, pt);
                pt = fma(f[10], c2, pt); pt = fma(f[11], s2, pt);
            } else {
                // polar form: one sine per product
                X = f[4] * sin_rev64(fma(-nz, p.z, f[5] - pxy));
                Y = f[6] * sin_rev64(fma(nz, p.z, f[7] - pxy));
            }
            const double sp = X + Y, sm = X - Y;
            fx = fma(nx, sp, fx);
            fy = fma(ny, sp, fy);
            fz = fma(nz, sm, fz);
            if (MODE == 2) {
                const double tx = wx * nx * sp, ty = wy * ny * sp, tz = wz * nz * sm;
                pt = fma(tx, tx, fma(ty, ty, fma(tz, tz, pt)));
            }
        }
        F.x = fma(wx, fx, F.x); F.y = fma(wy, fy, F.y); F.z = fma(wz, fz, F.z); F.w += pt;
    });
}

int choose_ksplit(int64_t nb, int P) {
    // split the k-loop across blocks when there are too few particles to fill the chip
    int split = 1;
    while (nb * split < 2048 && split * 2 <= 64 && (P + split * 2 - 1) / (split * 2) >= 8) split *= 2;
    return split;
}

hipError_t launch_kforce(rbe2d_ctx *h, const double *pos, const double *q, double *F, double *dEdq,
                         uint32_t flags, bool accumulate, bool want_pot, bool add_real, const double *gE,
                         hipStream_t s, const ForceExtra &x) {
    if (h->n_total == 0) return hipSuccess;
    ForceArgs a{};
    a.p32 = h->w.p32; a.p64 = h->w.p64; a.kn32 = h->w.kn32;
    a.kf32 = h->w.kf32; a.kf64 = h->w.kf64; a.lay = h->w.lay; a.sys = h->w.sys;
    a.n_sys = h->n_sys; a.P = h->P; a.P_pad = h->P_pad;
    a.pos = pos; a.q = q; a.scal = h->w.scal; a.real = real_parts(h);
    a.F = F; a.dEdq = dEdq; a.gE = gE; a.var = x.var;
    a.accumulate = accumulate; a.add_real = add_real; a.want_pot = want_pot; a.want_var = x.var != nullptr;
    a.do_kspace = (flags & RBE2D_KSPACE) != 0; a.do_ibc = (flags & RBE2D_IBC) != 0;
    a.split = 1;
    if (a.do_kspace) {
        a.split = h->force_ksplit ? h->force_ksplit
                                  : (h->tuned_now && h->tune.ksplit ? h->tune.ksplit : choose_ksplit(h->n_blocks, h->P));
        while (a.split > 1 && (int64_t)a.split * h->n_blocks > h->split_blocks) a.split >>= 1;
    }
    a.k_per_split = (h->P + a.split - 1) / a.split;
    const bool energies = x.energy || x.dEdgamma;
    const ForceSplit split = a.split == 1 ? kWhole : a.split > kMaxForceWaves && h->P > kLongP ? kRows : kWaves;
    if (energies) a.en = energy_args(h, x.energy, flags, gE, x.dEdgamma);
    a.err = h->w.err; a.err_out = x.err_out;
    a.n_groups = h->n_blocks * (kBlock / kWave);
    a.part = h->w.fpart; a.part_stride = (int64_t)h->n_blocks * kBlock;
    a.rows = split == kRows ? (a.split + kRowWaves - 1) / kRowWaves : 1;
    const int waves = split == kRows ? kRowWaves : std::min(a.split, kMaxForceWaves);
    const bool energies_ride = energies && split != kWhole && !timed(h, 6);
    const int energy_blocks = energies_ride ? h->n_sys : 0;
    const dim3 g(split == kWhole ? h->n_blocks : a.n_groups + (split == kWaves ? energy_blocks : 0), a.rows);
    const dim3 b(split == kWhole ? kBlock : waves * kWave);
    const int lds = split == kWhole ? 0 : waves * kWave * (int)sizeof(double4);
    const bool fp32 = h->precision == RBE2D_PREC_FP32_PHASE;
    const int mode = x.var ? 2 : want_pot ? 1 : 0;
    prof_begin(h, 5, s);
#define RBE2D_FORCE(M, S)                                                              \
    if (mode == M && split == S) {                                                     \
        if (fp32) hipLaunchKernelGGL((k_force32<M, S>), g, b, lds, s, a);              \
        else hipLaunchKernelGGL((k_force64<M, S>), g, b, lds, s, a);                   \
    }
    RBE2D_FORCE(0, kWhole) RBE2D_FORCE(1, kWhole) RBE2D_FORCE(2, kWhole)
    RBE2D_FORCE(0, kWaves) RBE2D_FORCE(1, kWaves) RBE2D_FORCE(2, kWaves)
    RBE2D_FORCE(0, kRows) RBE2D_FORCE(1, kRows) RBE2D_FORCE(2, kRows)
#undef RBE2D_FORCE
    if (split == kRows)
        hipLaunchKernelGGL(k_force_rows, dim3(h->n_blocks + energy_blocks), dim3(kBlock), 0, s, a, h->n_blocks);
    prof_end(h, 5, s);
    hipError_t e = hipGetLastError();
    // a launch of its own: the energies of an unsplit pass are a small part of the call
    if (e == hipSuccess && energies && !energies_ride) e = launch_energy(h, x.energy, flags, gE, x.dEdgamma, s);
    if (split != kWaves && e == hipSuccess && x.err_out) e = launch_copy_err(h, x.err_out, s);
    return e;
}

}  // namespace rbe2d
