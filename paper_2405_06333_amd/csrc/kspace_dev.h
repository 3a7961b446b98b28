// Device code of the k-space chain that other launches carry along too:
// structure factors and per-k assembly of small calls (kspace.hip).
#pragma once

#include "devmath.h"
#include "rbe2d_internal.h"

namespace rbe2d {

// Per-k records that are the same for a whole wave: read as constant memory
// they come by scalar loads also where the compiler cannot tell that the
// launch's other stores (the split force pass's LDS, the energies) leave them
// alone; as vector loads they took 40 more registers there.
typedef float vec4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) vec4f ConstFloat4;
typedef __attribute__((address_space(4))) double ConstDouble;
__device__ __forceinline__ float4 record(const float4 *p) {
    const vec4f v = *(const ConstFloat4 *)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ double4 record(const double4 *p) {
    const ConstDouble *v = (const ConstDouble *)p;
    return make_double4(v[0], v[1], v[2], v[3]);
}

// scal layout (kScal per system): 0 mu = sum q z, 1 Q = sum q, 2 sum q^2,
// 3 muM (image dipole of Theorem 3.3), 4 F_ibc,z / q_i, 5 offset of the
// IBC potential, 6 dmuM/dgamma_top, 7 dmuM/dgamma_bot, 8 S2 = sum q z^2;
// with surface charges (zero otherwise): F_z / q_i gains 10 + 9 z, the
// potential dE/dq_i gains 11 + 12 z + 13 z^2, the energy 14, and
// dE/dgamma_{top,bot} 15, 16
struct ScalArgs {
    const double *bpart;
    const SysDesc *sys;
    Layout lay;
    double *scal;
};

// IBC scalars of system r from the prep pass's block sums, by one wave
// (fixed summation order: the same in both launches that use it)
__device__ void ibc_scalars(const ScalArgs &a, int r, int lane) {
    const SysDesc &d = a.sys[r];
    double v[4] = {0, 0, 0, 0};
    for (int b = a.lay.bbase[r] + lane; b < a.lay.bbase[r + 1]; b += 64)
        for (int c = 0; c < 4; c++) v[c] += a.bpart[4 * b + c];
    for (int c = 0; c < 4; c++) v[c] = wave_sum(v[c]);
    if (lane == 0) {
        const double mu = v[0], Q = v[1], S2 = v[3];
        const double muM = d.g1 * mu + d.cgam * Q;
        const double tv = 2.0 * kPi / d.V * d.pref;
        double *o = a.scal + kScal * r;
        o[0] = mu;
        o[1] = Q;
        o[2] = v[2];
        o[3] = muM;
        o[4] = -tv * (muM + d.g1 * mu);
        o[5] = tv * mu * d.cgam;
        o[6] = d.dg1t * mu + d.dcgt * Q;
        o[7] = d.dg1b * mu + d.dcgb * Q;
        o[8] = S2;
        for (int c = 9; c < kScal; c++) o[c] = 0.0;
        if (d.surf) {
            // sheets: phi_s = -Es z + Cs; net charge: U_Q = -(tv / 2) Q (2 Gs S2 + 2 A1 mu + A0 Q)
            const double pe = d.pref;
            o[9] = 2.0 * tv * Q * d.Gs[0];
            o[10] = pe * d.Es[0] + tv * Q * d.A1[0];
            o[11] = pe * d.Cs[0] - tv * (d.Gs[0] * S2 + d.A1[0] * mu + d.A0[0] * Q);
            o[12] = -pe * d.Es[0] - tv * Q * d.A1[0];
            o[13] = -tv * Q * d.Gs[0];
            for (int k = 0; k < 3; k++) {
                const double e = -0.5 * tv * Q * (2.0 * d.Gs[k] * S2 + 2.0 * d.A1[k] * mu + d.A0[k] * Q) +
                                 pe * (-d.Es[k] * mu + d.Cs[k] * Q);
                o[k == 0 ? 14 : 14 + k] = e;
            }
        }
    }
}

// Blocks are dealt round-robin to the 8 XCDs.  Map block b to (tile, k-chunk)
// so that XCD b mod 8 runs all k-chunks of its tiles back to back: a tile is
// then fetched into one XCD's L2 once instead of once per k-chunk.  The grid
// has ceil(n_tiles / 8) * 8 * nkc blocks; blocks past the last tile exit.
struct TileChunk {
    int tile, kc;
};
__device__ __forceinline__ TileChunk tile_chunk(int b, int nkc) {
    const int j = b >> 3;
    return TileChunk{(j / nkc) * 8 + (b & 7), j % nkc};
}

struct SfArgs {
    const float4 *p32;
    const double4 *p64;
    const float4 *kn32;
    const double4 *kn64;
    const int *tbase;
    int n_sys, per, P_pad, n_tiles;   // per: particles per thread
    double *part;
};

// LDS of one structure-factor block
template <int KC>
struct SfLds32 {
    double sh[kBlock / 64][64];
};
template <int KC>
struct SfLds64 {
    double sh[kBlock / 64][4 * KC];
    double2 tab[kParts];
};

// Structure factors of one (tile, k-chunk) by kBlock threads (tid), which meet
// the same barriers as any other threads of their launch's block.  CONST: the
// k-vectors are read as constant memory (`record`), where the compiler does
// not find out by itself; in the launches of their own that form costs
// registers (FP64: 0.78 instead of 0.62 ms for 1e6 ions).

// FP32 phases and transcendentals; each thread sums its (at most 16)
// particles in FP32, and every sum after that -- across the 64 lanes, the
// waves of the block and (in the assembly) the tiles -- is in FP64.
template <int KC, bool CONST>
__device__ __forceinline__ void sf32_block(const float4 *__restrict__ p32, const float4 *__restrict__ kn,
                                           const int *tbase, int n_sys, int per_thread, int P_pad,
                                           double *__restrict__ part, TileChunk tc, int tid, double (&sh)[kBlock / 64][64]) {
    static_assert(4 * KC == 64, "one wave-transposed value per lane");
    const int r = find_sys(tbase, n_sys, tc.tile);
    const float4 *knr = kn + (int64_t)r * P_pad + tc.kc * KC;
    float acc[4 * KC];
#pragma unroll
    for (int v = 0; v < 4 * KC; v++) acc[v] = 0.0f;
    const int64_t base = (int64_t)tc.tile * kBlock * per_thread + tid;
    for (int m = 0; m < per_thread; m++) {
        const int64_t i = base + (int64_t)m * kBlock;
        const float4 u = p32[2 * i];
        const float4 w = p32[2 * i + 1];
#pragma unroll
        for (int kk = 0; kk < KC; kk++) {
            const float4 n = CONST ? record(knr + kk) : knr[kk];
            // nx fxh + ny fyh is exact (see the header comment)
            float pxy = fractf(fmaf(n.y, u.z, n.x * u.x));
            pxy = fmaf(n.x, u.y, pxy);
            pxy = fmaf(n.y, u.w, pxy);
            const float pz = fmaf(n.z, w.y, fractf(n.z * w.x));
            const float ph = pxy + pz, phh = pxy - pz;
            acc[4 * kk + 0] = fmaf(w.z, cos_rev(ph), acc[4 * kk + 0]);
            acc[4 * kk + 1] = fmaf(w.z, sin_rev(ph), acc[4 * kk + 1]);
            acc[4 * kk + 2] = fmaf(w.z, cos_rev(phh), acc[4 * kk + 2]);
            acc[4 * kk + 3] = fmaf(w.z, sin_rev(phh), acc[4 * kk + 3]);
        }
    }
    const int lane = tid & 63, wid = tid >> 6;
    // first butterfly stage of the wave transpose-reduce: the FP32 values are
    // exchanged, then widened and added in FP64; the other stages run in FP64
    double v[2 * KC];
    {
        const bool upper = (lane & 32) != 0;
#pragma unroll
        for (int i = 0; i < 2 * KC; i++) {
            const float send = upper ? acc[i] : acc[i + 2 * KC];
            const float keep = upper ? acc[i + 2 * KC] : acc[i];
            v[i] = (double)keep + (double)__shfl_xor(send, 32, 64);
        }
    }
    TransposeStage<KC, 2 * KC, double>::run(v, lane);
    sh[wid][lane] = v[0];
    __syncthreads();
    if (tid < 4 * KC) {
        double t = 0.0;
#pragma unroll
        for (int v2 = 0; v2 < kBlock / 64; v2++) t += sh[v2][tid];
        part[((int64_t)tc.tile * P_pad + tc.kc * KC) * 4 + tid] = t;
    }
}

// FP64: the phases' xy and z parts are taken separately, with e = q e^{2 pi i
// phi_xy} and z = 2 pi phi_z, into the four sums of (Re e, Im e) x (cos z, sin z)
// whose sums and differences are rho and rhohat.  The k-vectors come sorted by
// |nz| (k_ktable64), and sin z and cos z are kept from one to the next while
// |nz| stays the same; both come from the table of devmath.h.  Bound by VALU
// issue (0.98 of the slots): 26 instructions per (particle, k) and 20 more
// where |nz| changes, instead of 70 for two full sine-cosine pairs.  1e6 ions,
// P = 500, half of the |nz| repeated: 0.60 ms instead of 0.96.
template <int KC, bool CONST>
__device__ __forceinline__ void sf64_block(const double4 *__restrict__ p64, const double4 *__restrict__ ks,
                                           const int *tbase, int n_sys, int per_thread, int P_pad,
                                           double *__restrict__ part, TileChunk tc, int tid,
                                           double (&sh)[kBlock / 64][4 * KC], double2 (&tab)[kParts]) {
    if (tid < kParts) tab[tid] = make_double2(kPartTable[tid][0], kPartTable[tid][1]);
    __syncthreads();
    const int r = find_sys(tbase, n_sys, tc.tile);
    const double4 *ksr = ks + (int64_t)r * P_pad + tc.kc * KC;
    double acc[4 * KC];
#pragma unroll
    for (int v = 0; v < 4 * KC; v++) acc[v] = 0.0;
    const int64_t base = (int64_t)tc.tile * kBlock * per_thread + tid;
    for (int m = 0; m < per_thread; m++) {
        const double4 p = p64[base + (int64_t)m * kBlock];
        double sz, cz;
#pragma unroll
        for (int kk = 0; kk < KC; kk++) {
            const double4 n = CONST ? record(ksr + kk) : ksr[kk];
            if (kk == 0 || __double_as_longlong(n.z) != __double_as_longlong(CONST ? record(ksr + kk - 1).z : ksr[kk - 1].z))
                sincos_table64(n.z * p.z, tab, &sz, &cz);
            double s, c;
            sincos_table64(fma(n.y, p.y, n.x * p.x), tab, &s, &c);
            const double qc = p.w * c, qs = p.w * s;
            acc[4 * kk + 0] = fma(qc, cz, acc[4 * kk + 0]);
            acc[4 * kk + 1] = fma(qs, sz, acc[4 * kk + 1]);
            acc[4 * kk + 2] = fma(qs, cz, acc[4 * kk + 2]);
            acc[4 * kk + 3] = fma(qc, sz, acc[4 * kk + 3]);
            // keeps the sums of this k ahead of the next one's branch (the
            // compiler gathers them at the end otherwise, with 182 registers)
            asm volatile("" : "+v"(acc[4 * kk]), "+v"(acc[4 * kk + 1]), "+v"(acc[4 * kk + 2]), "+v"(acc[4 * kk + 3]));
        }
    }
    const int lane = tid & 63, wid = tid >> 6;
    wave_transpose_reduce<4 * KC>(acc, lane);
    if (lane < 4 * KC) sh[wid][lane] = acc[0];
    __syncthreads();
    if (tid < 4 * KC) {
        // rho (re, im) and rhohat (re, im) of one k; for nz < 0 the two change places
        const int kk = tid >> 2, v = tid & 3;
        const double id = ksr[kk].w;    // +-(1 + index in the k-set), the sign of nz; 0: padding
        if (id != 0.0) {
            const int l = (int)fabs(id) - 1;
            double t = 0.0, u = 0.0;
#pragma unroll
            for (int w = 0; w < kBlock / 64; w++) {
                t += sh[w][4 * kk + 2 * (v & 1)];
                u += sh[w][4 * kk + 2 * (v & 1) + 1];
            }
            // rho: cc - ss, sc + cs; rhohat: cc + ss, sc - cs
            const bool hat = (v >= 2) != (id < 0.0);
            part[((int64_t)tc.tile * P_pad + l) * 4 + v] = hat == ((v & 1) != 0) ? t - u : t + u;
        }
    }
}

struct AssembleArgs {
    const double *part;         // structure-factor partials [tile][P_pad][4], FP64 in both precisions
    int P, P_pad;
    const int *tbase;
    const int32_t *kset;
    const SysDesc *sys;
    const ImgTable *img;
    double *krec;
    float4 *kf32;
    double *kf64;              // FP64: the force pass's records
    int n_sys, with_scalars;   // with_scalars: n_sys more blocks compute the IBC scalars
    ScalArgs sc;
    long long *step;           // MD step counter to advance, or null
    int items() const { return n_sys * P + (with_scalars ? n_sys : 0); }   // waves
};

__device__ __forceinline__ double dmono(int e_self, double g_self, int e_other, double g_other) {
    // d/dg_self of g_self^e_self g_other^e_other
    if (e_self == 0) return 0.0;
    double r = (double)e_self;
    for (int i = 0; i < e_self - 1; i++) r *= g_self;
    for (int i = 0; i < e_other; i++) r *= g_other;
    return r;
}

// a double held by lane `src`, read by every lane
__device__ __forceinline__ double lane_value(double v, int src) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                            __builtin_amdgcn_readlane(__double2loint(v), src));
}

// One wave per (system, k), and with_scalars one more per system: wave number
// `item`.  DG: also the gamma derivatives of Y_odd and Y_even (for dE/dgamma;
// zero otherwise).
template <bool DG>
__device__ __forceinline__ void assemble_wave(const AssembleArgs &a, int item, int lane) {
    if (item >= a.n_sys * a.P) {
        const int r = item - a.n_sys * a.P;
        if (r >= a.n_sys || !a.with_scalars) return;
        ibc_scalars(a.sc, r, lane);
        if (a.step && r == 0 && lane == 0) *a.step += 1;
        return;
    }
    const int r = item / a.P, l = item - r * a.P;
    const SysDesc &d = a.sys[r];
    const ImgTable &it = a.img[r];
    // v[0..3]: this lane's share of rho and rhohat (lanes split the tiles);
    // v[4..7]: Yo, Ye; v[8..15]: dYo/dg_top, dYe/dg_top, dYo/dg_bot,
    // dYe/dg_bot (lanes split the image orders o = lane+1, lane+65, ...)
    constexpr int NV = DG ? 16 : 8;
    double v[NV];
#pragma unroll
    for (int c = 0; c < NV; c++) v[c] = 0.0;
    for (int t = a.tbase[r] + lane; t < a.tbase[r + 1]; t += 64) {
        const int64_t o = ((int64_t)t * a.P_pad + l) * 4;
        for (int c = 0; c < 4; c++) v[c] += a.part[o + c];
    }
    const int64_t kg = (int64_t)r * a.P + l;
    const int nx = a.kset[3 * kg], ny = a.kset[3 * kg + 1], nz = a.kset[3 * kg + 2];
    const double rev_per_H = (double)nz * d.H / d.Lz;   // kz H / (2 pi)
    for (int o = lane + 1; o <= d.M; o += 64) {
        const double gpl = it.gp[o - 1], gml = it.gm[o - 1];
        double mp, mm;   // multiples of kz H in the exponents of the + and - terms
        int slot;
        if (o & 1) { mp = (double)(o + 1); mm = -(double)(o - 1); slot = 4; }
        else       { mp = (double)o;       mm = -(double)o;       slot = 6; }
        double sp, cp, sm, cm;
        sincos_rev64(mp * rev_per_H, &sp, &cp);
        sincos_rev64(mm * rev_per_H, &sm, &cm);
        v[slot] += gpl * cp + gml * cm;
        v[slot + 1] += gpl * sp + gml * sm;
        if constexpr (DG) {
            const double dpt = dmono(it.ea_p[o - 1], d.g_top, it.eb_p[o - 1], d.g_bot);
            const double dmt = dmono(it.ea_m[o - 1], d.g_top, it.eb_m[o - 1], d.g_bot);
            const double dpb = dmono(it.eb_p[o - 1], d.g_bot, it.ea_p[o - 1], d.g_top);
            const double dmb = dmono(it.eb_m[o - 1], d.g_bot, it.ea_m[o - 1], d.g_top);
            v[4 + slot] += dpt * cp + dmt * cm;
            v[5 + slot] += dpt * sp + dmt * sm;
            v[8 + slot] += dpb * cp + dmb * cm;
            v[9 + slot] += dpb * sp + dmb * sm;
        }
    }
    // the NV wave sums at once (fixed-order butterfly): lane c then holds
    // the sum of value c, which every lane reads
    wave_transpose_reduce<NV>(v, lane);
    double S[NV];
#pragma unroll
    for (int c = 0; c < NV; c++) S[c] = lane_value(v[0], c);
    const double rr = S[0], ri = S[1], hr = S[2], hi = S[3];
    const double *y = S + 4;   // Yo, Ye (re, im), then the derivatives
    const double kx = 2.0 * kPi * nx / d.Lx, ky = 2.0 * kPi * ny / d.Ly, kz = 2.0 * kPi * nz / d.Lz;
    const double k2 = kx * kx + ky * ky + kz * kz;
    const double c = d.cfac / k2;
    // rho^M = (1 + Ye) rho + Yo rhohat
    const double er = 1.0 + y[2], ei = y[3];
    const double mr = er * rr - ei * ri + y[0] * hr - y[1] * hi;
    const double mi = er * ri + ei * rr + y[0] * hi + y[1] * hr;
    // A = rho^M + (1 + conj Ye) rho ; B = conj(Yo) rho
    const double Ar = mr + er * rr + ei * ri;
    const double Ai = mi + er * ri - ei * rr;
    const double Br = y[0] * rr + y[1] * ri;
    const double Bi = y[0] * ri - y[1] * rr;
    // polar form for the force passes, Im(e^{-i ph} cA) = |cA| sin(arg cA - ph):
    // lane 1 for A, lane 2 for B, in parallel
    constexpr double inv2pi = 0.15915494309189535;
    double mag = 0.0, arg = 0.0;
    if (lane == 1 || lane == 2) {
        const double xr = lane == 1 ? Ar : Br, xi = lane == 1 ? Ai : Bi;
        mag = c * hypot(xr, xi);
        arg = atan2(xi, xr) * inv2pi;
    }
    const double magA = lane_value(mag, 1), argA = lane_value(arg, 1);
    const double magB = lane_value(mag, 2), argB = lane_value(arg, 2);
    if (lane != 0) return;
    const double e = c * (rr * mr + ri * mi);
    // d e / d gamma = c Re(rho conj(dYe rho + dYo rhohat))
    double de[2] = {0.0, 0.0};
    if constexpr (DG) {
        for (int w = 0; w < 2; w++) {
            const double *dy = y + 4 + 4 * w;
            const double tr = dy[2] * rr - dy[3] * ri + dy[0] * hr - dy[1] * hi;
            const double ti = dy[2] * ri + dy[3] * rr + dy[0] * hi + dy[1] * hr;
            de[w] = c * (rr * tr + ri * ti);
        }
    }
    double *rec = a.krec + kg * kKRec;
    rec[0] = e; rec[1] = de[0]; rec[2] = de[1];
    if (a.kf64) {
        double *f = a.kf64 + kg * kKF64;
        f[0] = nx; f[1] = ny; f[2] = nz;
        f[4] = magA; f[5] = argA; f[6] = magB; f[7] = argB;
        f[8] = c * Ar; f[9] = c * Ai; f[10] = c * Br; f[11] = c * Bi;
        return;
    }
    a.kf32[3 * kg] = make_float4((float)kx, (float)ky, (float)kz, (float)(kx * kx + ky * ky));
    a.kf32[3 * kg + 1] = make_float4((float)(c * Ar), (float)(c * Ai), (float)(c * Br), (float)(c * Bi));
    a.kf32[3 * kg + 2] = make_float4((float)magA, (float)argA, (float)magB, (float)argB);
}

ScalArgs scal_args(rbe2d_ctx *h);
SfArgs sf_args(rbe2d_ctx *h);
AssembleArgs assemble_args(rbe2d_ctx *h, bool with_scalars, long long *step);
hipError_t launch_assemble(rbe2d_ctx *h, const AssembleArgs &a, bool want_dg, hipStream_t s);
// FP64 pair sums, with the assembly when `as` is set
void launch_tile_pairs(rbe2d_ctx *h, bool want_dg, const AssembleArgs *as, hipStream_t s);

}  // namespace rbe2d
