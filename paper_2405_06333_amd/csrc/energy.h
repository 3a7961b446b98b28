// Energies of all systems, as blocks of the launch that ends a force call or
// in a launch of their own.
#pragma once

#include "devmath.h"
#include "rbe2d_internal.h"

namespace rbe2d {

// energy components {total, real, kspace, self, ibc} per system and, in
// backward mode, gE * dE/dgamma_{top,bot}.  One block per system, fixed
// summation order.
struct EnergyArgs {
    const double *krec, *scal;
    const double *rpart;     // real-space sums per wave, in `parts` parts `stride` waves apart
    int parts, stride;
    const SysDesc *sys;
    Layout lay;
    int P;
    int do_real, do_k, do_ibc, want_dg;
    double *energy;          // 5 per system
    const double *gE;
    double *dEdgamma;        // 2 per system
};

// sh: blockDim.x / 64 doubles
__device__ __forceinline__ void energy_block(const EnergyArgs &a, int r, double *sh) {
    const SysDesc &d = a.sys[r];
    double ek = 0.0, dkt = 0.0, dkb = 0.0, er = 0.0, drt = 0.0, drb = 0.0;
    if (a.do_k)
        for (int l = threadIdx.x; l < a.P; l += (int)blockDim.x) {
            const double *rec = a.krec + ((int64_t)r * a.P + l) * kKRec;
            ek += rec[0];
            dkt += rec[1];
            dkb += rec[2];
        }
    const bool has_real = a.do_real && a.lay.off[r + 1] > a.lay.off[r];
    if (has_real)
        for (int p = 0; p < a.parts; p++) {
            const double *rp = a.rpart + (int64_t)3 * p * a.stride;
            for (int wv = a.lay.sbase[r] / kWave + threadIdx.x; wv < a.lay.sbase[r + 1] / kWave; wv += (int)blockDim.x) {
                er += rp[3 * wv];
                drt += rp[3 * wv + 1];
                drb += rp[3 * wv + 2];
            }
        }
    ek = block_sum(ek, sh);
    er = block_sum(er, sh);
    if (a.want_dg) {
        dkt = block_sum(dkt, sh); dkb = block_sum(dkb, sh);
        drt = block_sum(drt, sh); drb = block_sum(drb, sh);
    }
    if (threadIdx.x != 0) return;
    const double *sc = a.scal + kScal * r;
    const double tv = 2.0 * kPi / d.V * d.pref;
    const double Er = has_real ? 0.5 * er : 0.0;
    const double Ek = a.do_k ? ek : 0.0;
    const double Es = a.do_k ? -d.alpha * d.pref / sqrt(kPi) * sc[2] : 0.0;
    const double Ei = a.do_ibc ? tv * sc[0] * sc[3] + sc[14] : 0.0;   // sc[14]: surface terms (or 0)
    if (a.energy) {
        double *o = a.energy + 5 * r;
        o[0] = Er + Ek + Es + Ei;
        o[1] = Er;
        o[2] = Ek;
        o[3] = Es;
        o[4] = Ei;
    }
    if (a.want_dg && a.dEdgamma) {
        const double g = a.gE ? a.gE[r] : 1.0;
        const double ibt = a.do_ibc ? tv * sc[0] * sc[6] + sc[15] : 0.0;
        const double ibb = a.do_ibc ? tv * sc[0] * sc[7] + sc[16] : 0.0;
        a.dEdgamma[2 * r] = g * ((has_real ? 0.5 * drt : 0.0) + (a.do_k ? dkt : 0.0) + ibt);
        a.dEdgamma[2 * r + 1] = g * ((has_real ? 0.5 * drb : 0.0) + (a.do_k ? dkb : 0.0) + ibb);
    }
}

inline EnergyArgs energy_args(rbe2d_ctx *h, double *energy, uint32_t flags, const double *gE, double *dEdgamma) {
    EnergyArgs a;
    a.krec = h->w.krec; a.rpart = h->real_parts > 1 ? h->w.rpart_s : h->w.rpart; a.scal = h->w.scal; a.sys = h->w.sys; a.lay = h->w.lay;
    a.P = h->P; a.parts = h->real_parts; a.stride = h->real_stride;
    a.do_real = (flags & RBE2D_REAL) != 0;
    a.do_k = (flags & RBE2D_KSPACE) != 0;
    a.do_ibc = (flags & RBE2D_IBC) != 0;
    a.want_dg = dEdgamma != nullptr;
    a.energy = energy; a.gE = gE; a.dEdgamma = dEdgamma;
    return a;
}

}  // namespace rbe2d
