// Mixed-precision particle passes: SPH density (eq. sdpd-rho-v) with the
// active-pair masks, and the conservative pressure forces (eq. cons-forces),
// from FP32 positions relative to each particle's cell (ModelF32 of
// neighbours.hpp).  Kernel values and the per-particle sums are FP32; rho, f,
// eps and everything downstream (the equation of state, the F/D update, the
// observables) stay FP64.
#include "neighbours.hpp"

namespace sdpd {

__device__ __forceinline__ void density_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_body<ModelF32, true>(a, blk);
}
__device__ __forceinline__ void density_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_body<ModelF32, false>(a, blk);
}
__device__ __forceinline__ void forces_lucy_body(const ForcesArgs &a, uint32_t blk)
{
    forces_body<ModelF32, true>(a, blk);
}
__device__ __forceinline__ void forces_cubic_body(const ForcesArgs &a, uint32_t blk)
{
    forces_body<ModelF32, false>(a, blk);
}
__device__ __forceinline__ void density_sparse_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_sparse<ModelF32, true>(a, blk);
}
__device__ __forceinline__ void density_dense_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_dense<ModelF32, true>(a, blk);
}
__device__ __forceinline__ void density_sparse_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_sparse<ModelF32, false>(a, blk);
}
__device__ __forceinline__ void density_dense_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_dense<ModelF32, false>(a, blk);
}
SDPD_MULTI_KERNEL(k_density_f32_sparse_lucy_multi, DensityArgs, density_sparse_lucy_body, 256)
SDPD_MULTI_KERNEL(k_density_f32_dense_lucy_multi, DensityArgs, density_dense_lucy_body, 64,
                  ModelF32::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_f32_sparse_cubic_multi, DensityArgs, density_sparse_cubic_body, 256)
SDPD_MULTI_KERNEL(k_density_f32_dense_cubic_multi, DensityArgs, density_dense_cubic_body, 64,
                  ModelF32::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_f32_lucy_multi, DensityArgs, density_lucy_body, 64 * kCellWaves,
                  ModelF32::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_f32_cubic_multi, DensityArgs, density_cubic_body, 64 * kCellWaves,
                  ModelF32::kDensityOcc)
SDPD_MULTI_KERNEL(k_forces_f32_lucy_multi, ForcesArgs, forces_lucy_body, 256)
SDPD_MULTI_KERNEL(k_forces_f32_cubic_multi, ForcesArgs, forces_cubic_body, 256)

// P_i / rho_i^2 into the w slot of the particle's FP32 record
struct PressureF32Args {
    DevParams P;
    const double *eps, *rho;
    float *q4f;
};
__device__ __forceinline__ void pressure_term_f32_body(const PressureF32Args &a, uint32_t blk)
{
    int64_t i = (int64_t)blk * blockDim.x + threadIdx.x;
    if (i < a.P.n) a.q4f[4 * i + 3] = (float)(a.P.cPi * a.eps[i] / a.rho[i]);
}
__global__ void k_pressure_term_f32(PressureF32Args a) { pressure_term_f32_body(a, blockIdx.x); }
SDPD_MULTI_KERNEL(k_pressure_term_f32_multi, PressureF32Args, pressure_term_f32_body, 256)

int run_density_f32(sdpd_ctx *c, const sdpd_state *s, int update_eps)
{
    timer_begin(c, TK_DENSITY);
    const DensityArgs args{c->dp, c->q4f, c->cell_sorted, c->cell_start, s->rho, s->eps,
                           update_eps, c->masks, c->list, c->list_count, c->list_len,
                           c->list_cap, c->err, nullptr, density_reach2(c->dp), c->dense};
    const DensityMulti lucy{k_density_f32_lucy_multi, k_density_f32_sparse_lucy_multi,
                            k_density_f32_dense_lucy_multi};
    const DensityMulti cubic{k_density_f32_cubic_multi, k_density_f32_sparse_cubic_multi,
                             k_density_f32_dense_cubic_multi};
    const int rc = c->dp.kernel == SDPD_KERNEL_LUCY ? launch_density<ModelF32, true>(c, args, lucy)
                                                    : launch_density<ModelF32, false>(c, args, cubic);
    timer_end(c, TK_DENSITY);
    return rc;
}

int run_forces_f32(sdpd_ctx *c, const sdpd_state *s, int half_kick)
{
    timer_begin(c, TK_FORCE);
    int rc = launch_or_record(c, k_pressure_term_f32, k_pressure_term_f32_multi,
                              (unsigned)((c->n + 255) / 256), 256, 0,
                              PressureF32Args{c->dp, s->eps, s->rho, c->q4f});
    const ForcesArgs args{partner_args(c, c->q4f), s->f, s->p, half_kick};
    if (!rc)
        rc = c->dp.kernel == SDPD_KERNEL_LUCY
                 ? launch_forces<ModelF32, true>(c, args, k_forces_f32_lucy_multi)
                 : launch_forces<ModelF32, false>(c, args, k_forces_f32_cubic_multi);
    timer_end(c, TK_FORCE);
    return rc;
}

}  // namespace sdpd
