// On-device k-sampler: the same draws as the host sampler in api.hip; the
// k-set of system r uses stream id (stream_base + r), where stream_base is
// the argument or, for graph replays, n_sys times a device step counter.
#pragma once

#include "rbe2d_internal.h"

namespace rbe2d {

struct SampleArgs {
    const double *cdf;
    const SysDesc *sys;
    int n_sys, P;
    uint64_t seed, stream_base;
    const long long *dev_step;   // if set: stream_base = n_sys * (*dev_step)
    int32_t *kset;
    int *err;
};

inline SampleArgs sample_args(rbe2d_ctx *h, uint64_t seed, uint64_t stream_id, const long long *dev_step) {
    SampleArgs a;
    a.cdf = h->w.cdf; a.sys = h->w.sys; a.n_sys = h->n_sys; a.P = h->P;
    a.seed = seed; a.stream_base = stream_id; a.dev_step = dev_step;
    a.kset = h->w.kset; a.err = h->w.err;
    return a;
}

// k-vector l of system r
__device__ __forceinline__ int3 draw_kvec(const SampleArgs &a, int r, int l) {
    const SysDesc &d = a.sys[r];
    const uint64_t base = a.dev_step ? (uint64_t)(*a.dev_step) * (uint64_t)a.n_sys : a.stream_base;
    const uint64_t key = stream_key(a.seed, base + (uint64_t)r);
    for (int att = 0; att < 64; att++) {
        const uint64_t c = ((uint64_t)l * 64 + att) * 3;
        const int nx = draw_axis(a.cdf + d.cdf_off[0], d.nmax[0], uniform01(key, c));
        const int ny = draw_axis(a.cdf + d.cdf_off[1], d.nmax[1], uniform01(key, c + 1));
        const int nz = draw_axis(a.cdf + d.cdf_off[2], d.nmax[2], uniform01(key, c + 2));
        if (nx | ny | nz) return make_int3(nx, ny, nz);
    }
    atomicOr(a.err, 2);
    return make_int3(1, 0, 0);
}

}  // namespace rbe2d
