// Adjoint (reverse-mode gradient) of the conservative SDPD dynamics: the
// Velocity-Verlet steps of eq. (sdpd-verlet) with the SPH density of
// eq. (sdpd-rho-v), the constant-entropy energy update of Sec. 3.1 and the
// pressure force of eq. (cons-forces); the F/D sweep is off.
//
// With the entropies fixed by the initial state, eps_k = c_k rho_k^g with
// g = A kB / Cv and c_k = eps0_k rho0_k^-g, so P_k / rho_k^2 = Pi_k =
// kap c_k rho_k^(g-1), kap = A kB / (m Cv).  One step maps (q, p) to
//   p' = p + h f(q),  q'' = q + dt p'/m,  p'' = p' + h f(q''),  h = dt/2,
// so the cotangents go back as
//   lq += h Jf(q'')^T lp,  lp += (dt/m) lq,  lq += h Jf(q)^T lp,
// and the product Jf(q^n)^T (h lp^n) serves the second half kick of step
// n - 1 and the first of step n: one product per configuration.  With
// v = h lp, for the pairs (i, j) within h (r = q_i - q_j, u = v_i - v_j):
//   pibar_k  = m^2 sum_j F(r_kj) (r_kj . u_kj)              cotangent of Pi_k
//   rhobar_k = pibar_k (g - 1) Pi_k / rho_k                 through Pi(rho)
//   qbar_i   = sum_j m^2 (Pi_i + Pi_j) [F u + (F'/r)(r . u) r]
//              - m (rhobar_i + rhobar_j) F r                through rho(q)
// (grad W = -F r).  The products accumulate G_k = sum pibar_k Pi_k and
// H_k = sum pibar_k Pi_k ln rho_k, which give the initial-state path
// (rho0bar = -g G / rho0 through the density of q0, eps0bar = G / eps0)
// and dJ/dA = sum_k G_k / A + (kB/Cv)(H_k - G_k ln rho0_k).  The reference
// density rho0 cancels (eps depends on eps0 and rho / rho0_k only).
//
// Cotangents of the final energies and densities (J may read eps_K, rho_K,
// e.g. the mean pressure of the closure of Sec. 2.1.2): since
// eps_K = c rho_K^g, epsbar_K adds g epsbar eps_K / rho_K to rhobar_K, which
// together with the caller's rhobar_K enters the density term of the final
// configuration's q product, and epsbar eps_K to the cotangent of ln c
// (Ge), which joins G on the initial-state path; its A part is
// (kB/Cv)(He - Ge ln rho0) with He = Ge ln rho_K (no 1/A term: eps has no
// A prefactor).  The conservative dynamics depends on A and Cv only through
// A/Cv (g = A kB/Cv, kap = A kB/(m Cv)), so at fixed A
// dJ/dCv = -(A/Cv) dJ/dA for a J without an explicit Cv dependence.
//
// Forward: checkpoints of the full state every `every` steps; backward:
// each segment is recomputed from its checkpoint (bit-identical: the same
// kernels on the same data), its configurations kept, and processed in
// reverse.  Cotangents live in id order (ids must be 0..n-1).
#include <math.h>

#include <algorithm>

#include <new>
#include <type_traits>
#include <utility>
#include <vector>

#include "neighbours.hpp"

namespace sdpd {

constexpr int kSumBlocks = 256;   // blocks of the dA sum (and threads of its last one)

struct StateBuf {
    double *q = nullptr, *p = nullptr, *eps = nullptr, *rho = nullptr, *f = nullptr;
    uint32_t *id = nullptr;
    sdpd_state view() const { return sdpd_state{q, p, eps, rho, f, id}; }
};

struct AdjointWork {
    int K = 0, every = 0, nck = 0;
    std::vector<StateBuf> ckpt, seg;
    double *lq = nullptr, *lp = nullptr, *G = nullptr, *H = nullptr;   // id order
    double *Ge = nullptr, *He = nullptr;   // final-energy path (id order)
    double *eps0 = nullptr, *rho0 = nullptr;                             // id order
    double4 *v4 = nullptr;       // (v, Pi), cell order
    double *rhobar = nullptr;    // cell order
    double *partial = nullptr;   // sums of dA: per block, then the total
    uint32_t *idcount = nullptr;
    void *base = nullptr;        // all of it: one allocation, kept for the next forward pass
    size_t bytes = 0;
};

void adjoint_free(AdjointWork *a)
{
    if (!a) return;
    if (a->base) (void)hipFree(a->base);
    delete a;
}

// the buffers one after the other from base on (NULL: only their size)
static size_t adjoint_layout(AdjointWork *a, size_t n, char *base)
{
    size_t used = 0;
    auto place = [&](auto *&p, size_t count) {
        p = reinterpret_cast<typename std::remove_reference<decltype(p)>::type>(base + used);
        used += (sizeof(*p) * count + 255) / 256 * 256;
    };
    auto state = [&](StateBuf &s) {
        place(s.q, 3 * n);
        place(s.p, 3 * n);
        place(s.f, 3 * n);
        place(s.eps, n);
        place(s.rho, n);
        place(s.id, n);
    };
    for (auto &s : a->ckpt) state(s);
    for (auto &s : a->seg) state(s);
    place(a->v4, n);
    for (double **p : {&a->lq, &a->lp}) place(*p, 3 * n);
    for (double **p : {&a->G, &a->H, &a->Ge, &a->He, &a->eps0, &a->rho0, &a->rhobar}) place(*p, n);
    place(a->partial, kSumBlocks + 1);
    place(a->idcount, n);
    return used;
}

// dst = src, every array of the state
struct StateCopy {
    StateBuf dst, src;
};
__global__ __launch_bounds__(256) void k_copy_state(int64_t n, StateCopy c)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    double v[11];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        v[x] = c.src.q[x * n + k];
        v[3 + x] = c.src.p[x * n + k];
        v[6 + x] = c.src.f[x * n + k];
    }
    v[9] = c.src.eps[k];
    v[10] = c.src.rho[k];
    const uint32_t id = c.src.id[k];
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        c.dst.q[x * n + k] = v[x];
        c.dst.p[x * n + k] = v[3 + x];
        c.dst.f[x * n + k] = v[6 + x];
    }
    c.dst.eps[k] = v[9];
    c.dst.rho[k] = v[10];
    c.dst.id[k] = id;
}

static int copy_state(sdpd_ctx *c, const StateBuf &dst, const sdpd_state &src)
{
    const StateBuf s{src.q, src.p, src.eps, src.rho, src.f, src.id};
    hipLaunchKernelGGL(k_copy_state, dim3((unsigned)((c->n + 255) / 256)), dim3(256), 0, c->stream,
                       c->n, StateCopy{dst, s});
    return check_hip(hipGetLastError());
}

// dJ/dA = sum of G / A + kB/Cv (H - G ln rho0 + He - Ge ln rho0): sums of kSumBlocks
// blocks (first launch), then of those (second, one block, into partial[kSumBlocks])
struct SumArgs {
    int64_t n;
    const double *G, *H, *Ge, *He, *rho0;
    double inv_A, kc;
    double *partial;
    int last;
};
__global__ __launch_bounds__(256) void k_sum_dA(SumArgs a)
{
    __shared__ double s[256];
    double v = 0.0;
    if (a.last) {
        v = a.partial[threadIdx.x];
    } else {
        for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < a.n;
             k += (int64_t)kSumBlocks * 256) {
            const double l = log(a.rho0[k]);
            v += a.G[k] * a.inv_A + a.kc * (a.H[k] - a.G[k] * l) + a.kc * (a.He[k] - a.Ge[k] * l);
        }
    }
    s[threadIdx.x] = v;
    for (int off = 128; off > 0; off >>= 1) {
        __syncthreads();
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
    }
    if (threadIdx.x == 0) a.partial[a.last ? kSumBlocks : blockIdx.x] = s[0];
}

// ---------------------------------------------------------------- kernels

__global__ void k_count_ids(int64_t n, const uint32_t *id, uint32_t *count, uint32_t *err)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint32_t i = id[k];
    if (i >= (uint64_t)n) {
        atomicOr(err, ERR_IDS);
        return;
    }
    if (atomicAdd(&count[i], 1u) != 0u) atomicOr(err, ERR_IDS);
}

__global__ void k_axpy(int64_t len, double a, const double *x, double *y)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < len) y[k] += a * x[k];
}

// state value (cell order) -> id order
__global__ void k_to_id(int64_t n, const uint32_t *id, const double *src, double *dst)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) dst[id[k]] = src[k];
}

// v = (h lp, Pi) per particle in cell order
__global__ void k_pack_v(DevParams P, const uint32_t *id, const double *lp, const double *eps,
                         const double *rho, double4 *v4)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= P.n) return;
    const int64_t i = id[k];
    const double h = 0.5 * P.dt;
    double4 r;
    r.x = h * lp[i];
    r.y = h * lp[P.n + i];
    r.z = h * lp[2 * P.n + i];
    r.w = P.cPi * eps[k] / rho[k];
    v4[k] = r;
}

// rhobar into the w slots of the position records (id: rhobar in id order)
__global__ void k_pack_rhobar(int64_t n, const uint32_t *id, const double *rhobar, double *q4)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) q4[4 * k + 3] = rhobar[id ? id[k] : k];
}

// F (r . u)
template <bool LUCY>
struct PiTerm {
    const DevParams &P;
    const double4 *__restrict__ v4;
    double4 v;
    __device__ __forceinline__ void at(int64_t i) { v = v4[i]; }
    __device__ __forceinline__ void operator()(uint32_t j, bool own, const double4 &,
                                               const double4 &, const double d[3], double r2,
                                               double out[1]) const
    {
        const double4 u = v4[j];
        const double ru = d[0] * (v.x - u.x) + d[1] * (v.y - u.y) + d[2] * (v.z - u.z);
        double v1 = ModelF64::force<LUCY>(P, r2) * ru;
        asm volatile("" : "+v"(v1));   // (as in the forces)
        out[0] = own ? 0.0 : v1;
    }
};

// m^2 (Pi_i + Pi_j) [F u + (F'/r)(r . u) r] - m (rhobar_i + rhobar_j) F r over cF;
// without the first part if !FORCE
template <bool LUCY, bool FORCE>
struct QTerm {
    const DevParams &P;
    const double4 *__restrict__ v4;
    double4 v;
    __device__ __forceinline__ void at(int64_t i) { if (FORCE) v = v4[i]; }
    __device__ __forceinline__ void operator()(uint32_t j, bool own, const double4 &qi,
                                               const double4 &qj, const double d[3], double r2,
                                               double out[3]) const
    {
        // r^2 + DBL_MIN: r^2 for every distinct pair; finite, and times zero, for r = 0
        const double y = fast_rsq(r2 + DBL_MIN), x = r2 * y * P.inv_h, t = 1.0 - x;
        double F, dFr;   // F, F'/r
        if (LUCY) {
            F = t * t;
            dFr = -2.0 * t * P.inv_h * y;
        } else if (x <= 0.5) {
            F = 2.0 - 3.0 * x;
            dFr = -3.0 * P.inv_h * y;
        } else {
            F = P.h * (t * t) * y;
            dFr = -P.h * (1.0 - x * x) * (y * y) * y;
        }
        const double sr = -P.m * (qi.w + qj.w) * F;
        for (int c = 0; c < 3; ++c) out[c] = sr * d[c];
        if (FORCE) {
            const double4 vj = v4[j];
            const double u[3] = {v.x - vj.x, v.y - vj.y, v.z - vj.z};
            const double Pij = P.m * P.m * (v.w + vj.w);
            const double ru = (d[0] * u[0] + d[1] * u[1] + d[2] * u[2]) * dFr;
            for (int c = 0; c < 3; ++c) out[c] += Pij * (F * u[c] + ru * d[c]);
        }
        for (int c = 0; c < 3; ++c) out[c] = own ? 0.0 : out[c];
    }
};

// rhobar (cell order, also into the w slots of q4); G, H accumulate (id order) with
// the weight
template <bool LUCY>
__global__ __launch_bounds__(256) void k_vjp_pi(PartnerArgs a, const double4 *v4,
                                                const double *__restrict__ rho,
                                                const uint32_t *__restrict__ id, double weight,
                                                double *rhobar, double *q4, double *G, double *H)
{
    const DevParams &P = a.P;
    bool live;
    const int64_t i = partner_particle<ModelF64>(P, xcd_block(blockIdx.x, gridDim.x), live);
    const int lane = threadIdx.x & 63;
    PartnerSums<ModelF64, 1, PiTerm<LUCY>> sums{a, P, nullptr, lane,
                                                (uint32_t)lane % ModelF64::kLanes};
    const double acc = sums.run(i, live, PiTerm<LUCY>{P, v4, double4()});
    if (!live || sums.s != 0u) return;
    const double pb = P.m * P.m * P.cF * acc, Pi = v4[i].w;
    const double rb = pb * (P.eps_exp - 1.0) * Pi / rho[i];
    rhobar[i] = rb;
    q4[4 * i + 3] = rb;
    const int64_t g = id[i];
    G[g] += weight * pb * Pi;
    H[g] += weight * pb * Pi * log(rho[i]);
}

// lq (id order) += weight * qbar: the density term, and the force term (FORCE)
template <bool LUCY, bool FORCE>
__global__ __launch_bounds__(256) void k_vjp_q(PartnerArgs a, const double4 *v4,
                                               const uint32_t *__restrict__ id, double weight,
                                               double *lq)
{
    const DevParams &P = a.P;
    bool live;
    const int64_t i = partner_particle<ModelF64>(P, xcd_block(blockIdx.x, gridDim.x), live);
    const int lane = threadIdx.x & 63;
    PartnerSums<ModelF64, 3, QTerm<LUCY, FORCE>> sums{a, P, nullptr, lane,
                                                      (uint32_t)lane % ModelF64::kLanes};
    const double w = sums.run(i, live, QTerm<LUCY, FORCE>{P, v4, double4()});
    if (live && sums.s < 3u) lq[sums.s * P.n + id[i]] += weight * (P.cF * w);
}

// cotangents of the final energies and densities (id order, either may be
// NULL) at the final configuration (cell order): rhobar += drho + g deps
// eps / rho, Ge = deps eps, He = Ge ln rho
__global__ void k_final_cotangent(int64_t n, double g, const uint32_t *id, const double *deps,
                                  const double *drho, const double *eps, const double *rho,
                                  double *rhobar, double *Ge, double *He)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int64_t i = id[k];
    const double de = deps ? deps[i] : 0.0;
    const double dr = drho ? drho[i] : 0.0;
    rhobar[k] += dr + g * de * eps[k] / rho[k];
    const double ge = de * eps[k];
    Ge[i] = ge;
    He[i] = ge * log(rho[k]);
}

// (G + Ge) -> eps0bar = (G + Ge) / eps0 and rho0bar = -g (G + Ge) / rho0
// (id order, into the given outputs)
__global__ void k_initial_path(int64_t n, double g, const double *G, const double *Ge,
                               const double *eps0, const double *rho0, double *eps0bar,
                               double *rho0bar)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double gt = G[k] + Ge[k];
    if (eps0bar) eps0bar[k] = gt / eps0[k];
    rho0bar[k] = -g * gt / rho0[k];
}

static inline unsigned nblk(int64_t n) { return (unsigned)((n + 255) / 256); }

// one vector-Jacobian product of the force at configuration X (already in
// W): lq += weight * Jf(q)^T (h lp), G and H accumulate.  At the final
// configuration (weight 1) the cotangents of the final energies and
// densities (deps, drho: id order, may be NULL) join the density term.
static int vjp_config(sdpd_ctx *c, AdjointWork *a, const sdpd_state &Ws, double weight,
                      const double *deps = nullptr, const double *drho = nullptr)
{
    const int64_t n = c->n;
    int rc;
    if ((rc = run_build_cells(c, &Ws, 0))) return rc;
    if ((rc = run_density(c, &Ws, 0))) return rc;
    const bool lucy = c->dp.kernel == SDPD_KERNEL_LUCY;
    const PartnerArgs pa = partner_args(c, c->q4);
    hipLaunchKernelGGL(k_pack_v, dim3(nblk(n)), dim3(256), 0, c->stream, c->dp, Ws.id, a->lp,
                       Ws.eps, Ws.rho, a->v4);
    hipLaunchKernelGGL(lucy ? k_vjp_pi<true> : k_vjp_pi<false>, dim3(nblk(ModelF64::kLanes * n)), dim3(256),
                       0, c->stream, pa, a->v4, Ws.rho, Ws.id, weight, a->rhobar, c->q4, a->G,
                       a->H);
    if (deps || drho) {
        hipLaunchKernelGGL(k_final_cotangent, dim3(nblk(n)), dim3(256), 0, c->stream, n,
                           c->dp.eps_exp, Ws.id, deps, drho, Ws.eps, Ws.rho, a->rhobar, a->Ge,
                           a->He);
        hipLaunchKernelGGL(k_pack_rhobar, dim3(nblk(n)), dim3(256), 0, c->stream, n,
                           (const uint32_t *)nullptr, a->rhobar, c->q4);
    }
    hipLaunchKernelGGL((lucy ? k_vjp_q<true, true> : k_vjp_q<false, true>), dim3(nblk(ModelF64::kLanes * n)),
                       dim3(256), 0, c->stream, pa, a->v4, Ws.id, weight, a->lq);
    return check_hip(hipGetLastError());
}

}  // namespace sdpd

using namespace sdpd;

extern "C" {

int sdpd_adjoint_forward(sdpd_ctx *c, sdpd_state *s, int nsteps, int every)
{
    if (!c || !s || nsteps < 1 || every < 1 || !c->cells_valid) return SDPD_EINVAL;
    if (c->prm.fd != SDPD_FD_NONE || c->prm.prec != SDPD_FP64 || c->n == 0) return SDPD_EINVAL;
    if (!s->q || !s->p || !s->eps || !s->rho || !s->f || !s->id) return SDPD_EINVAL;
    const int64_t n = c->n;
    // the last pass's memory serves this one if it is large enough, and no more than
    // twice what is needed
    AdjointWork *a = new (std::nothrow) AdjointWork();
    if (!a) return SDPD_ENOMEM;
    a->K = nsteps;
    a->every = every;
    a->nck = (nsteps + every - 1) / every;
    a->ckpt.resize(a->nck);
    a->seg.resize(every + 1);
    const size_t need = adjoint_layout(a, (size_t)n, nullptr);
    if (c->adj && c->adj->bytes >= need && c->adj->bytes / 2 <= need) {
        std::swap(a->base, c->adj->base);
        a->bytes = c->adj->bytes;
    }
    adjoint_free(c->adj);
    c->adj = nullptr;
    if (!a->base) {
        if (hipMalloc(&a->base, need) != hipSuccess) {
            a->base = nullptr;
            (void)hipGetLastError();
            adjoint_free(a);
            return SDPD_ENOMEM;
        }
        a->bytes = need;
    }
    adjoint_layout(a, (size_t)n, static_cast<char *>(a->base));
    int rc = SDPD_OK;
    c->adj = a;
    // ids must be a permutation of 0..n-1 (cotangents are indexed by id)
    if ((rc = launch_fill_u32(c, a->idcount, 0u, n))) return rc;
    hipLaunchKernelGGL(k_count_ids, dim3(nblk(n)), dim3(256), 0, c->stream, n, s->id, a->idcount,
                       c->err);
    hipLaunchKernelGGL(k_to_id, dim3(nblk(n)), dim3(256), 0, c->stream, n, s->id, s->eps,
                       a->eps0);
    hipLaunchKernelGGL(k_to_id, dim3(nblk(n)), dim3(256), 0, c->stream, n, s->id, s->rho,
                       a->rho0);
    if ((rc = check_hip(hipGetLastError()))) return rc;
    for (int k = 0; k < nsteps; ++k) {
        if (k % every == 0 && (rc = copy_state(c, a->ckpt[k / every], *s))) return rc;
        if ((rc = enqueue_step(c, s, (uint64_t)k, true))) return rc;
    }
    return SDPD_OK;
}

}  // extern "C"

namespace sdpd {

// reverse pass from the cotangents of the final state (q, p: 3 x n; eps,
// rho: n; id order; q, p required, eps, rho may be NULL); dA and dCv (host,
// may be NULL) synchronise
static int adjoint_backward(sdpd_ctx *c, const double *dJ_dq, const double *dJ_dp,
                            const double *dJ_deps, const double *dJ_drho, double *dJ_dq0,
                            double *dJ_dp0, double *dJ_deps0, double *dJ_dA, double *dJ_dCv)
{
    AdjointWork *a = c->adj;
    const int64_t n = c->n;
    const size_t d3 = sizeof(double) * 3 * (size_t)n;
    int rc = SDPD_OK;
    if ((rc = check_hip(hipMemcpyAsync(a->lq, dJ_dq, d3, hipMemcpyDeviceToDevice, c->stream))))
        return rc;
    if ((rc = check_hip(hipMemcpyAsync(a->lp, dJ_dp, d3, hipMemcpyDeviceToDevice, c->stream))))
        return rc;
    for (double *z : {a->G, a->H, a->Ge, a->He})
        if ((rc = launch_fill_u64(c, (unsigned long long *)z, 0ull, n))) return rc;
    const double dt_m = c->prm.dt / c->prm.m;
    for (int sg = a->nck - 1; sg >= 0; --sg) {
        const int start = sg * a->every, end = std::min(start + a->every, a->K);
        // recompute the segment's configurations start .. end
        if ((rc = copy_state(c, a->seg[0], a->ckpt[sg].view()))) return rc;
        for (int k = 1; k <= end - start; ++k) {
            const sdpd_state cur = a->seg[k - 1].view();
            if ((rc = copy_state(c, a->seg[k], cur))) return rc;
            const sdpd_state nxt = a->seg[k].view();
            if ((rc = enqueue_step(c, &nxt, (uint64_t)(start + k - 1), true))) return rc;
        }
        if (sg == a->nck - 1) {   // the final configuration: second half kick of step K-1
            if ((rc = vjp_config(c, a, a->seg[end - start].view(), 1.0, dJ_deps, dJ_drho)))
                return rc;
        }
        for (int N = end - 1; N >= start; --N) {
            hipLaunchKernelGGL(k_axpy, dim3(nblk(3 * n)), dim3(256), 0, c->stream, 3 * n, dt_m,
                               a->lq, a->lp);
            // (its state is not needed again: the product sorts it in place)
            if ((rc = vjp_config(c, a, a->seg[N - start].view(), N > 0 ? 2.0 : 1.0))) return rc;
        }
    }
    // initial-state path: the entropies come from eps0 and rho(q0)
    const double g = c->dp.eps_exp;
    double *eps0bar = dJ_deps0;
    hipLaunchKernelGGL(k_initial_path, dim3(nblk(n)), dim3(256), 0, c->stream, n, g, a->G, a->Ge,
                       a->eps0, a->rho0, eps0bar, a->rhobar);   // rhobar: id order here
    // the last product left configuration 0 with its cells and lists
    const sdpd_state Ws = a->seg[0].view();
    hipLaunchKernelGGL(k_pack_rhobar, dim3(nblk(n)), dim3(256), 0, c->stream, n, Ws.id, a->rhobar,
                       c->q4);
    hipLaunchKernelGGL((c->dp.kernel == SDPD_KERNEL_LUCY ? k_vjp_q<true, false>
                                                         : k_vjp_q<false, false>),
                       dim3(nblk(ModelF64::kLanes * n)), dim3(256), 0, c->stream, partner_args(c, c->q4),
                       a->v4, Ws.id, 1.0, a->lq);
    if ((rc = check_hip(hipGetLastError()))) return rc;
    if ((rc = check_hip(hipMemcpyAsync(dJ_dq0, a->lq, d3, hipMemcpyDeviceToDevice, c->stream))))
        return rc;
    if ((rc = check_hip(hipMemcpyAsync(dJ_dp0, a->lp, d3, hipMemcpyDeviceToDevice, c->stream))))
        return rc;
    if (dJ_dA || dJ_dCv) {
        SumArgs s{n, a->G, a->H, a->Ge, a->He, a->rho0, 1.0 / c->dp.A, c->prm.kB / c->prm.Cv,
                  a->partial, 0};
        hipLaunchKernelGGL(k_sum_dA, dim3(kSumBlocks), dim3(256), 0, c->stream, s);
        s.last = 1;
        hipLaunchKernelGGL(k_sum_dA, dim3(1), dim3(256), 0, c->stream, s);
        if ((rc = check_hip(hipGetLastError()))) return rc;
        double acc = 0.0;
        if ((rc = check_hip(hipMemcpyAsync(&acc, a->partial + kSumBlocks, sizeof acc,
                                           hipMemcpyDeviceToHost, c->stream))))
            return rc;
        if ((rc = check_hip(hipStreamSynchronize(c->stream)))) return rc;
        if (dJ_dA) *dJ_dA = acc;
        if (dJ_dCv) *dJ_dCv = -(c->dp.A / c->prm.Cv) * acc;
    }
    return SDPD_OK;
}

}  // namespace sdpd

extern "C" {

int sdpd_adjoint_backward(sdpd_ctx *c, const double *dJ_dq, const double *dJ_dp, double *dJ_dq0,
                          double *dJ_dp0, double *dJ_deps0, double *dJ_dA)
{
    if (!c || !c->adj || !dJ_dq || !dJ_dp || !dJ_dq0 || !dJ_dp0) return SDPD_EINVAL;
    return adjoint_backward(c, dJ_dq, dJ_dp, nullptr, nullptr, dJ_dq0, dJ_dp0, dJ_deps0, dJ_dA,
                            nullptr);
}

int sdpd_adjoint_vjp(sdpd_ctx *c, const sdpd_cotangent *ct, sdpd_gradient *gr)
{
    if (!c || !c->adj || !ct || !gr || !ct->dq || !ct->dp || !gr->dq0 || !gr->dp0)
        return SDPD_EINVAL;
    gr->dA = gr->dCv = gr->drho0 = 0.0;
    int rc = adjoint_backward(c, ct->dq, ct->dp, ct->deps, ct->drho, gr->dq0, gr->dp0, gr->deps0,
                              &gr->dA, &gr->dCv);
    if (!rc) rc = check_hip(hipStreamSynchronize(c->stream));
    gr->drho0 = 0.0;   // rho0 cancels from the dynamics (eps depends on rho/rho0_k only)
    return rc;
}

}  // extern "C"
