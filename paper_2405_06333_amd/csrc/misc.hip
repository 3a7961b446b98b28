// Small launches of their own: energies, k-draws, the MD step counter, the
// error word.
#include "devmath.h"
#include "energy.h"
#include "rbe2d_internal.h"
#include "sampler.h"

namespace rbe2d {

// ---------------------------------------------------------------------------
// energies (energy.h) in a launch of their own: where no force pass follows
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_energy(EnergyArgs a) {
    __shared__ double sh[kBlock / 64];
    energy_block(a, blockIdx.x, sh);
}

hipError_t launch_energy(rbe2d_ctx *h, double *energy, uint32_t flags, const double *gE, double *dEdgamma,
                         hipStream_t s) {
    const EnergyArgs a = energy_args(h, energy, flags, gE, dEdgamma);
    prof_begin(h, 6, s);
    hipLaunchKernelGGL(k_energy, dim3(h->n_sys), dim3(kBlock), 0, s, a);
    prof_end(h, 6, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// on-device k-sampler (sampler.h) in a launch of its own
// ---------------------------------------------------------------------------

__global__ void k_sample(SampleArgs a) {
    const int kg = blockIdx.x * blockDim.x + threadIdx.x;
    if (kg >= a.n_sys * a.P) return;
    const int r = kg / a.P;
    const int3 n = draw_kvec(a, r, kg - r * a.P);
    int32_t *k = a.kset + 3 * (int64_t)kg;
    k[0] = n.x; k[1] = n.y; k[2] = n.z;
}

hipError_t launch_sample(rbe2d_ctx *h, uint64_t seed, uint64_t stream_id, const long long *dev_step,
                         hipStream_t s) {
    const int n = h->n_sys * h->P;
    prof_begin(h, 8, s);
    hipLaunchKernelGGL(k_sample, dim3((n + 63) / 64), dim3(64), 0, s, sample_args(h, seed, stream_id, dev_step));
    prof_end(h, 8, s);
    return hipGetLastError();
}

__global__ void k_set_step(long long *step, long long v) { *step = v; }

hipError_t launch_set_step(rbe2d_ctx *h, long long value, hipStream_t s) {
    hipLaunchKernelGGL(k_set_step, dim3(1), dim3(1), 0, s, h->w.step, value);
    return hipGetLastError();
}

__global__ void k_copy_err(const int *src, int32_t *dst) {
    if (threadIdx.x == 0) *dst = *src;
}
hipError_t launch_copy_err(rbe2d_ctx *h, int32_t *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_err, dim3(1), dim3(64), 0, s, h->w.err, dst);
    return hipGetLastError();
}

}  // namespace rbe2d
