// SPH density, eq. (sdpd-rho-v), the entropy-conserving energy update of
// Sec. 3.1, and the active-pair masks of the fluctuation/dissipation sweep
// (FP64; the loops are in neighbours.hpp).
#include "neighbours.hpp"

namespace sdpd {

__device__ __forceinline__ void density_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_body<ModelF64, true>(a, blk);
}
__device__ __forceinline__ void density_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_body<ModelF64, false>(a, blk);
}
__device__ __forceinline__ void density_sparse_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_sparse<ModelF64, true>(a, blk);
}
__device__ __forceinline__ void density_dense_lucy_body(const DensityArgs &a, uint32_t blk)
{
    density_dense<ModelF64, true>(a, blk);
}
__device__ __forceinline__ void density_sparse_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_sparse<ModelF64, false>(a, blk);
}
__device__ __forceinline__ void density_dense_cubic_body(const DensityArgs &a, uint32_t blk)
{
    density_dense<ModelF64, false>(a, blk);
}
SDPD_MULTI_KERNEL(k_density_sparse_lucy_multi, DensityArgs, density_sparse_lucy_body, 256)
SDPD_MULTI_KERNEL(k_density_dense_lucy_multi, DensityArgs, density_dense_lucy_body, 64,
                  ModelF64::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_sparse_cubic_multi, DensityArgs, density_sparse_cubic_body, 256)
SDPD_MULTI_KERNEL(k_density_dense_cubic_multi, DensityArgs, density_dense_cubic_body, 64,
                  ModelF64::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_lucy_multi, DensityArgs, density_lucy_body, 64 * kCellWaves,
                  ModelF64::kDensityOcc)
SDPD_MULTI_KERNEL(k_density_cubic_multi, DensityArgs, density_cubic_body, 64 * kCellWaves,
                  ModelF64::kDensityOcc)

int run_density(sdpd_ctx *c, const sdpd_state *s, int update_eps, bool pack_rho)
{
    if (c->n == 0) {
        c->masks_valid = 1;
        return SDPD_OK;
    }
    if (c->dp.mixed) {
        const int rc = run_density_f32(c, s, update_eps);
        if (!rc) c->masks_valid = 1;
        return rc;
    }
    timer_begin(c, TK_DENSITY);
    const DensityArgs args{c->dp, c->q4, c->cell_sorted, c->cell_start, s->rho, s->eps,
                           update_eps, c->masks, c->list, c->list_count, c->list_len,
                           c->list_cap, c->err, pack_rho ? c->q4 : nullptr,
                           density_reach2(c->dp), c->dense};
    const DensityMulti lucy{k_density_lucy_multi, k_density_sparse_lucy_multi, k_density_dense_lucy_multi};
    const DensityMulti cubic{k_density_cubic_multi, k_density_sparse_cubic_multi, k_density_dense_cubic_multi};
    const int rc = c->dp.kernel == SDPD_KERNEL_LUCY ? launch_density<ModelF64, true>(c, args, lucy)
                                                    : launch_density<ModelF64, false>(c, args, cubic);
    timer_end(c, TK_DENSITY);
    if (!rc) c->masks_valid = 1;
    return rc;
}

}  // namespace sdpd
