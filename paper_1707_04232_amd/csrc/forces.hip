// Conservative pressure forces, eq. (cons-forces), fused with the second
// half kick of eq. (sdpd-verlet); observables (Sec. 2.2.1).
#include "neighbours.hpp"

#include <algorithm>

namespace sdpd {

// P_i / rho_i^2 from the ideal-gas closure: A kB rho eps / (m Cv) / rho^2
// Pi_i = P_i / rho_i^2, stored with the position as (x, y, z, Pi) so that
// the force pass reads one 32-byte record per partner
struct PressureArgs {
    DevParams P;
    const double *q, *eps, *rho;
    double *q4;
};
__device__ __forceinline__ void pressure_term_body(const PressureArgs &a, uint32_t blk)
{
    const DevParams &P = a.P;
    const double *q = a.q, *eps = a.eps, *rho = a.rho;
    double *q4 = a.q4;
    int64_t i = (int64_t)blk * blockDim.x + threadIdx.x;
    if (i >= P.n) return;
    const double v = P.cPi * eps[i] / rho[i];
    double4 r;
    r.x = q[i];
    r.y = q[P.n + i];
    r.z = q[2 * P.n + i];
    r.w = v;
    reinterpret_cast<double4 *>(q4)[i] = r;
}
__global__ void k_pressure_term(PressureArgs a) { pressure_term_body(a, blockIdx.x); }
SDPD_MULTI_KERNEL(k_pressure_term_multi, PressureArgs, pressure_term_body, 256)

// f_i = sum_{j != i, r < h} m^2 (Pi_i + Pi_j) F_ij r_ij over the partners
// listed by the density pass (same positions); optionally p_i += dt/2 f_i.
__device__ __forceinline__ void forces_lucy_body(const ForcesArgs &a, uint32_t blk)
{
    forces_body<ModelF64, true>(a, blk);
}
__device__ __forceinline__ void forces_cubic_body(const ForcesArgs &a, uint32_t blk)
{
    forces_body<ModelF64, false>(a, blk);
}
SDPD_MULTI_KERNEL(k_forces_lucy_multi, ForcesArgs, forces_lucy_body, 256)
SDPD_MULTI_KERNEL(k_forces_cubic_multi, ForcesArgs, forces_cubic_body, 256)

int run_forces(sdpd_ctx *c, const sdpd_state *s, int half_kick)
{
    if (c->n == 0) return SDPD_OK;
    if (c->dp.mixed) return run_forces_f32(c, s, half_kick);
    const unsigned g = (unsigned)((c->n + 255) / 256);
    timer_begin(c, TK_FORCE);
    int rc = launch_or_record(c, k_pressure_term, k_pressure_term_multi, g, 256, 0,
                              PressureArgs{c->dp, s->q, s->eps, s->rho, c->q4});
    const ForcesArgs args{partner_args(c, c->q4), s->f, s->p, half_kick};
    if (!rc)
        rc = c->dp.kernel == SDPD_KERNEL_LUCY
                 ? launch_forces<ModelF64, true>(c, args, k_forces_lucy_multi)
                 : launch_forces<ModelF64, false>(c, args, k_forces_cubic_multi);
    timer_end(c, TK_FORCE);
    return rc;
}

// --- observables: E_int, KE, P (3), min eps; deterministic two-level sums
constexpr int OBS_THREADS = 256;
constexpr int OBS_FIELDS = 6;

__global__ __launch_bounds__(OBS_THREADS) void k_observe_partial(DevParams P, const double *p,
                                                                 const double *eps,
                                                                 double *partial)
{
    __shared__ double s[OBS_FIELDS][OBS_THREADS];
    const int64_t n = P.n;
    double v[OBS_FIELDS] = {0.0, 0.0, 0.0, 0.0, 0.0, INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * OBS_THREADS + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * OBS_THREADS) {
        double px = p[i], py = p[n + i], pz = p[2 * n + i];
        v[0] += eps[i];
        v[1] += (px * px + py * py + pz * pz) / (2.0 * P.m);
        v[2] += px;
        v[3] += py;
        v[4] += pz;
        v[5] = fmin(v[5], eps[i]);
    }
    for (int k = 0; k < OBS_FIELDS; ++k) s[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int off = OBS_THREADS / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            for (int k = 0; k < 5; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + off];
            s[5][threadIdx.x] = fmin(s[5][threadIdx.x], s[5][threadIdx.x + off]);
        }
        __syncthreads();
    }
    if (threadIdx.x < OBS_FIELDS) partial[blockIdx.x * OBS_FIELDS + threadIdx.x] = s[threadIdx.x][0];
}


// one workgroup: partials summed in a fixed tree order (deterministic)
__global__ __launch_bounds__(OBS_THREADS) void k_observe_final(const double *partial,
                                                               int64_t nblocks,
                                                               const unsigned long long *counters,
                                                               double *rec)
{
    __shared__ double s[OBS_FIELDS][OBS_THREADS];
    double v[OBS_FIELDS] = {0.0, 0.0, 0.0, 0.0, 0.0, INFINITY};
    for (int64_t b = threadIdx.x; b < nblocks; b += OBS_THREADS) {
        for (int k = 0; k < 5; ++k) v[k] += partial[b * OBS_FIELDS + k];
        v[5] = fmin(v[5], partial[b * OBS_FIELDS + 5]);
    }
    for (int k = 0; k < OBS_FIELDS; ++k) s[k][threadIdx.x] = v[k];
    __syncthreads();
    for (int off = OBS_THREADS / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            for (int k = 0; k < 5; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + off];
            s[5][threadIdx.x] = fmin(s[5][threadIdx.x], s[5][threadIdx.x + off]);
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    rec[0] = s[0][0] + s[1][0];
    rec[1] = s[0][0];
    rec[2] = s[1][0];
    rec[3] = s[2][0];
    rec[4] = s[3][0];
    rec[5] = s[4][0];
    rec[6] = s[5][0];
    if (!counters) return;   // a record without the F/D counters (7 doubles)
    unsigned long long *ci = reinterpret_cast<unsigned long long *>(rec + 7);
    for (int k = 0; k < CNT_N; ++k) ci[k] = counters[k];
}

int observe_blocks(int64_t n) { return n > 0 ? (int)std::min<int64_t>(OBS_MAX_BLOCKS, (n + 255) / 256) : 0; }

int launch_observe(const DevParams &dp, const double *p, const double *eps, double *partial,
                   const unsigned long long *counters, double *dst_record, hipStream_t stream)
{
    const int nb = observe_blocks(dp.n);
    if (nb > 0)
        hipLaunchKernelGGL(k_observe_partial, dim3((unsigned)nb), dim3(OBS_THREADS), 0, stream,
                           dp, p, eps, partial);
    hipLaunchKernelGGL(k_observe_final, dim3(1), dim3(OBS_THREADS), 0, stream, partial,
                       (int64_t)nb, counters, dst_record);
    return check_hip(hipGetLastError());
}

int run_observe(sdpd_ctx *c, const sdpd_state *s, double *dst_record)
{
    return launch_observe(c->dp, s->p, s->eps, c->obs_partial, c->counters, dst_record,
                          c->stream);
}

}  // namespace sdpd
