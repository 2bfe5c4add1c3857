// Loops over the neighbour candidates and partners of a particle, shared by
// the FP64 and the FP32 (mixed precision) particle passes.
#pragma once

#include "sdpd_internal.hpp"
#include "fd_elem.hpp"

#include <float.h>

namespace sdpd {

// ---------------------------------------------------------------- arithmetic
// A model of the arithmetic: the type of positions and sums, the packed record
// (x, y, z and a scalar), the periodic shift of axis a for neighbour offset o
// (0, 1, 2) of a cell that is the first (lo) or the last (hi) of the axis, the
// active test and the terms.  Sums are formed in candidate order (offset index
// k = 0..26 with z slowest, then slot) in every form of a pass, so that the
// forms agree bit for bit.

// FP64: absolute positions; the image is chosen per neighbour cell: a cell
// reached across the box boundary contributes (x_i - x_j) +- L, which is the
// minimum-image difference for every pair closer than h (L >= 4 h), in the
// same rounding as the plain form.
struct ModelF64 {
    typedef double Real;
    typedef double4 Vec;
    static constexpr bool kShiftEverywhere = false;
    static constexpr int kChunks = 4, kEdgeChunks = 2;   // see DensityWave
    static __device__ __forceinline__ Real shift(const DevParams &P, int a, int o, bool lo, bool hi)
    {
        return o == 0 && lo ? P.box[a] : (o == 2 && hi ? -P.box[a] : 0.0);
    }
    static __device__ __forceinline__ bool near(const DevParams &P, Real r2) { return r2 < P.h2; }
    // W(r) over cW: W of Sec. 2.1.1 (Lucy's kernel or the cubic spline of
    // eq. sdpd-cubic-w) in t = 1 - r/h.  r = 0 (i itself): r^2 + DBL_MIN is r^2
    // for every other pair, exactly, and its root gives W(0).
    template <bool LUCY>
    static __device__ __forceinline__ Real density(const DevParams &P, Real r2)
    {
        const Real r = fd_sqrt(r2 + DBL_MIN);
        const Real t = fma(-P.inv_h, r, 1.0);
        if (LUCY) return t * t * t * fma(-3.0, t, 4.0);   // 1 + 3 x = 4 - 3 t
        const Real x = r * P.inv_h;
        return x <= 0.5 ? fma(-6.0 * x * x, t, 1.0) : 2.0 * (t * t * t);
    }
    static __device__ __forceinline__ double density_scale(const DevParams &P, Real acc)
    {
        return (P.m * P.cW) * acc;
    }
    // F(r) over cF with grad W(r) = -F(|r|) r (the spline's second branch is
    // 48/(pi h^4 r)(1 - r/h)^2); coincident particles: r^2 + DBL_MIN as above
    template <bool LUCY>
    static __device__ __forceinline__ Real force(const DevParams &P, Real r2)
    {
        const Real rsq = r2 + DBL_MIN;
        if (LUCY) {
            const Real t = fma(-P.inv_h, fd_sqrt(rsq), 1.0);
            return t * t;
        }
        const Real y = fast_rsq(rsq), x = rsq * y * P.inv_h, t = 1.0 - x;
        return x <= 0.5 ? fma(-3.0, x, 2.0) : P.h * (t * t) * y;
    }
    static __device__ __forceinline__ Real force_scale(const DevParams &P) { return P.m * P.m * P.cF; }
};

// FP32: positions relative to the particle's cell; the separation of particle
// i (cell c) and particle j of neighbour cell c + o is (xr_i - xr_j) - (o - 1)
// times the cell edge: no periodic case analysis and no loss of digits to the
// box size.
struct ModelF32 {
    typedef float Real;
    typedef float4 Vec;
    static constexpr bool kShiftEverywhere = true;
    static constexpr int kChunks = 3, kEdgeChunks = 3;
    static __device__ __forceinline__ Real shift(const DevParams &P, int a, int o, bool, bool)
    {
        return -(float)(o - 1) * P.cell_f[a];
    }
    static __device__ __forceinline__ bool near(const DevParams &P, Real r2) { return r2 < P.h2_f; }
    template <bool LUCY>
    static __device__ __forceinline__ Real density(const DevParams &P, Real r2)
    {
        const float x = sqrtf(r2) * P.inv_h_f, t = 1.0f - x;
        float w;
        if (LUCY) w = P.cW_f * (1.0f + 3.0f * x) * (t * t * t);
        else if (x <= 0.5f) w = P.cW_f * (1.0f - 6.0f * x * x + 6.0f * x * x * x);
        else w = 2.0f * P.cW_f * (t * t * t);
        return P.m_f * w;
    }
    static __device__ __forceinline__ double density_scale(const DevParams &, Real acc)
    {
        return (double)acc;
    }
    template <bool LUCY>
    static __device__ __forceinline__ Real force(const DevParams &P, Real r2)
    {
        const float r = sqrtf(r2), x = r * P.inv_h_f, t = 1.0f - x;
        if (LUCY) return P.cF_f * (t * t);
        if (x <= 0.5f) return P.cF_f * (2.0f - 3.0f * x);
        return P.cF_f * P.h_f * (t * t) / r;
    }
    static __device__ __forceinline__ Real force_scale(const DevParams &P) { return P.m_f * P.m_f; }
};

template <class M>
__device__ __forceinline__ typename M::Vec load_vec(const typename M::Real *q, int64_t j)
{
    return reinterpret_cast<const typename M::Vec *>(q)[j];
}

// LDS written by lanes of this wave is read by others of it after this point:
// a wave's LDS accesses complete in order, so only the compiler has to keep it
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct CellXyz {
    int x, y, z;
    __device__ __forceinline__ CellXyz(const DevParams &P, uint32_t c)
    {
        x = (int)(c % (uint32_t)P.nc[0]);
        y = (int)((c / (uint32_t)P.nc[0]) % (uint32_t)P.nc[1]);
        z = (int)(c / ((uint32_t)P.nc[0] * (uint32_t)P.nc[1]));
    }
};

// ---------------------------------------------------------------- cells
constexpr int kCellWaves = 4;      // waves, and cells, per workgroup

__device__ __forceinline__ uint32_t lane_of(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ double lane_of(double v, int l)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint64_t lo = lane_of((uint32_t)b, l), hi = lane_of((uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(hi << 32 | lo));
}
__device__ __forceinline__ float lane_of(float v, int l)
{
    return __uint_as_float(lane_of(__float_as_uint(v), l));
}
__device__ __forceinline__ uint32_t below(uint64_t ballot, uint32_t base)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, base));
}

// A wave's cell and its 27 neighbour cells (offset index k in lane k < 27).
// The particles of the neighbour cells, one cell after the other, are numbered
// 0 .. total - 1 ("positions"): the candidate order of the sums.
struct CellWave {
    NbSteps steps;
    uint32_t s, raw, cnt, b;   // lane k: first particle, particles, visited ones (0 in
                               // an overflowing cell), first position (lanes > 26: total)
    uint32_t own, m, total;    // first particle of the cell and its particles (visited)

    __device__ __forceinline__ CellWave(const DevParams &P, const CellXyz &cc,
                                        const uint32_t *cell_start)
        : steps(P, cc.x, cc.y, cc.z)
    {
        const int lane = threadIdx.x & 63;
        s = raw = 0u;
        if (lane < NNB) {
            const uint32_t cn = (uint32_t)steps.get(P, lane).c;
            s = cell_start[cn];
            raw = cell_start[cn + 1] - s;
        }
        cnt = raw > (uint32_t)P.cap ? 0u : raw;
        uint32_t incl = cnt;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
            if (lane >= off) incl += v;
        }
        total = lane_of(incl, NNB - 1);
        b = lane < NNB ? incl - cnt : total;
        own = lane_of(s, OWN_NB);
        m = lane_of(cnt, OWN_NB);
    }
    __device__ __forceinline__ bool edge() const { return (steps.lo | steps.hi) != 0u; }
    // cells k0 .. window(k0, limit) - 1 hold at most `limit` (>= 64) positions
    __device__ __forceinline__ int window(int k0, uint32_t limit) const
    {
        return __popcll(__ballot((threadIdx.x & 63u) < (uint32_t)NNB &&
                                 b + cnt <= lane_of(b, k0) + limit));
    }
    // the cell of position t < total and the particle there; called by the whole
    // wave (a lane that is switched off gives no value to the others)
    __device__ __forceinline__ void find(uint32_t t, int &k, uint32_t &j, uint32_t &slot) const
    {
        k = 0;
#pragma unroll
        for (int step = 16; step; step >>= 1)
            if ((uint32_t)__shfl((int)b, k + step) <= t) k += step;
        slot = t - (uint32_t)__shfl((int)b, k);
        j = (uint32_t)__shfl((int)s, k) + slot;
    }
};

// ---------------------------------------------------------------- density
struct DensityArgs {
    DevParams P;
    const void *q4;          // packed records of the model
    const uint32_t *cell_start;
    double *rho, *eps;
    int update_eps;
    uint64_t *masks;         // masks[k * n + i]: slot bits of the partners in cell k
    uint32_t *err;
    double *rho_w;           // FP64: also into the w slot of the record, or NULL
};

__device__ __forceinline__ void density_store(const DensityArgs &a, int64_t i, double rho)
{
    const double rho_old = a.rho[i];
    a.rho[i] = rho;
    // where the fluctuation/dissipation sweep of the step reads it (never read
    // in this pass)
    if (a.rho_w) a.rho_w[4 * i + 3] = rho;
    if (a.update_eps) {   // Sec. 3.1
        double e_new = a.eps[i] * pow(rho / rho_old, a.P.eps_exp);
        if (!(e_new > 0.0) || !isfinite(e_new)) atomicOr(a.err, ERR_NONFINITE);
        a.eps[i] = e_new;
    }
}

// Density and masks, one cell per wave.  The candidates sit in the lanes' registers,
// 64 K of them at a time (a window: whole neighbour cells); the wave goes through
// the cell's particles, tests its candidates against one of them at once, queues
// the squared distances in range in LDS, in candidate order, and evaluates the
// kernel for the queue at full lane occupancy; lane i then adds up the terms of
// particle i in order.  The test of particle i is bit i of a lane's word, which
// ends as the mask of its candidate for this cell: no pair is looked at twice
// and no mask is taken apart.
//
// Bound by the VALU: 460 candidates of a particle (17 per cell, h = 0.98 cell
// edges) take 7.2 lane-parallel tests of 14 instructions.  A thread per particle
// reads 24 B of every candidate through the L1 instead and runs to the largest
// cell of its wave: 677 us for 1M particles in FP64 (now 512), 3590 us for 8M in
// FP32 (now 2830), 251 us for 262k (now 169).
//
// K: more candidates per lane mean fewer windows, each with its own pass over the
// particles, and fewer waves per SIMD.  1M particles, K = 3, 4, 5, 8: 547, 515,
// 562, 864 us; 8M in FP32, K = 3, 4, 5: 2826, 2940, 3477.  FP64 cells at the
// boundary carry shifts (three doubles more per candidate) and take K = 2 (K = 4
// there: 532 us), or 4 where a wave per SIMD is all there is (SPLIT: 25 us
// against 28 for 8064 particles).
constexpr int kTerms = 832;        // queue entries of a wave
constexpr int kTail = 256;         // particles of a workgroup's shared last part

template <class M, bool SPLIT>
struct DensityLds {
    typename M::Real terms[kCellWaves][kTerms + 64];
    double rho[kTail];
    uint32_t words[SPLIT ? kCellWaves : 1][SPLIT ? 64 * kCellWaves : 1];
};

// SPLIT: the workgroup's waves share one cell, wave w with the particles in
// slots w q .. w q + q - 1 (q = ceil(m / 4)) of it, and put their words together
// in LDS: for boxes of so few cells that a wave per cell leaves SIMDs idle and the
// pass takes as long as one wave's chain (1000 particles: 18 us, a wave per cell
// 34, four lanes per particle 66)
template <class M, bool LUCY, bool SPLIT>
struct DensityWave {
    typedef typename M::Real Real;
    const DensityArgs &a;
    const DevParams &P;
    const CellWave &cw;
    DensityLds<M, SPLIT> &lds;
    const int lane, wave, lo, hi;   // slots lo .. hi - 1 are this wave's
    Real *terms;
    Real x, y, z, acc;       // lane i < m: particle i of the cell and its sum
    uint32_t beg, end;       // ... its terms in the queue
    uint32_t fill;

    // the queued squared distances to terms, and each lane's added to its sum
    __device__ __forceinline__ void flush()
    {
        wave_sync();
        for (uint32_t e = lane; e < fill; e += 64u) {
            const Real r2 = terms[e];
            const Real w = M::template density<LUCY>(P, r2);
            terms[e] = r2 < (Real)0 ? (Real)0 : w;
        }
        wave_sync();
        for (uint32_t r = beg; r < end; r += 4u) {
            Real v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = terms[r + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = acc + v[u];
        }
        wave_sync();
        fill = beg = end = 0u;
    }

    template <bool SHIFT, int K>
    __device__ __forceinline__ void window(uint32_t base, uint32_t width)
    {
        const Real *__restrict__ q4 = static_cast<const Real *>(a.q4);
        const int chunks = (int)((width + 63u) / 64u);
        Real cx[K], cy[K], cz[K], sh[K][3];
        uint32_t at[K];          // the candidate
        uint32_t self[K];        // k << 8 | slot
#pragma unroll
        for (int c = 0; c < K; ++c) {
            cx[c] = cy[c] = cz[c] = (Real)0;
            at[c] = self[c] = 0u;
            for (int d = 0; d < 3; ++d) sh[c][d] = (Real)0;
            if (c >= chunks) continue;
            const uint32_t t = 64u * c + lane;
            int k;
            uint32_t j, slot;
            cw.find(base + min(t, width - 1u), k, j, slot);   // (every lane takes part)
            const typename M::Vec v = load_vec<M>(q4, j);
            // a lane past the end: out of range of everything
            cx[c] = t < width ? v.x : (Real)1e18;
            cy[c] = v.y;
            cz[c] = v.z;
            at[c] = j;
            self[c] = (uint32_t)k << 8 | slot;
            if (SHIFT) {
                const int o[3] = {k % 3, (k / 3) % 3, k / 9};
                for (int d = 0; d < 3; ++d)
                    sh[c][d] = M::shift(P, d, o[d], (cw.steps.lo >> d) & 1u,
                                        (cw.steps.hi >> d) & 1u);
            }
        }
        const int m = (int)cw.m;
        for (int half = m > 32 ? 1 : 0; half >= 0; --half) {
            uint32_t w[K];
#pragma unroll
            for (int c = 0; c < K; ++c) w[c] = 0u;
            const int first_slot = max(lo, 32 * half);
            for (int i = min(hi, 32 * half + 32) - 1; i >= first_slot; --i) {
                const Real xi = lane_of(x, i), yi = lane_of(y, i), zi = lane_of(z, i);
                if (fill + 64u * K + 3u > (uint32_t)kTerms) flush();
                const uint32_t first = fill;
                Real *const unused = terms + kTerms + lane;
#pragma unroll
                for (int c = 0; c < K; ++c) {
                    if (c >= chunks) break;
                    Real dx = xi - cx[c], dy = yi - cy[c], dz = zi - cz[c];
                    if (SHIFT) {
                        dx += sh[c][0];
                        dy += sh[c][1];
                        dz += sh[c][2];
                    }
                    const Real r2 = dx * dx + dy * dy + dz * dz;
                    const bool near = M::near(P, r2);
                    const uint64_t hit = __ballot(near);
                    w[c] = w[c] + w[c] + (near ? 1u : 0u);
                    // (no branch: the other lanes write to slots that nothing reads)
                    uint32_t off = below(hit, 0u);
                    asm volatile("" : "+v"(off));   // (computed, not branched around)
                    *(near ? terms + fill + off : unused) = r2;
                    fill += (uint32_t)__popcll(hit);
                }
                // up to a multiple of four with entries without a term
                if (lane < 3) terms[fill + lane] = (Real)-1;
                fill = (fill + 3u) & ~3u;
                if (lane == i) {
                    beg = first;
                    end = fill;
                }
            }
            // lane j's word: the partners of candidate j in this cell
            if (SPLIT) {
                __syncthreads();   // (the last words have been read)
#pragma unroll
                for (int c = 0; c < K; ++c)
                    lds.words[wave][64 * c + lane] = w[c] << ((first_slot - 32 * half) & 31);
                __syncthreads();
            }
            uint32_t *words = reinterpret_cast<uint32_t *>(a.masks);
#pragma unroll
            for (int c = 0; c < K; ++c) {
                if (SPLIT && c != wave) continue;
                if (c < chunks && 64u * c + lane < width) {
                    const uint32_t k = self[c] >> 8, slot = self[c] & 255u;
                    uint32_t v = w[c];
                    if (SPLIT) {
                        v = 0u;
                        for (int o = 0; o < kCellWaves; ++o) v |= lds.words[o][64 * c + lane];
                    }
                    // i itself is no partner
                    if (k == (uint32_t)OWN_NB && (slot >> 5) == (uint32_t)half)
                        v &= ~(1u << (slot & 31u));
                    const int64_t e = (int64_t)((uint32_t)(NNB - 1) - k) * P.n + at[c];
                    if (m > 32) words[2 * e + half] = v;
                    else a.masks[e] = v;
                }
            }
        }
    }

    template <bool SHIFT, int K>
    __device__ __forceinline__ void windows()
    {
        for (int k0 = 0; k0 < NNB;) {
            const int k1 = cw.window(k0, 64u * K);
            const uint32_t base = lane_of(cw.b, k0), width = lane_of(cw.b, k1) - base;
            window<SHIFT, K>(base, width);
            flush();   // (a lane has one segment of the queue at a time)
            k0 = k1;
        }
    }

    __device__ __forceinline__ void run()
    {
        terms = lds.terms[wave];
        x = y = z = acc = (Real)0;
        beg = end = fill = 0u;
        if ((uint32_t)lane < cw.m) {
            const typename M::Vec v =
                load_vec<M>(static_cast<const Real *>(a.q4), cw.own + (uint32_t)lane);
            x = v.x;
            y = v.y;
            z = v.z;
        }
        if (!M::kShiftEverywhere && cw.edge()) windows<true, SPLIT ? M::kChunks : M::kEdgeChunks>();
        else windows<M::kShiftEverywhere, M::kChunks>();
        // overflowing cells: reported, not visited
        uint64_t over = __ballot(cw.raw != cw.cnt);
        if (over && lane == 0) atomicOr(a.err, ERR_CELLCAP);
        for (; over; over &= over - 1ull) {
            const int k = __builtin_ctzll(over);
            const uint32_t s = lane_of(cw.s, k), cnt = lane_of(cw.raw, k);
            for (uint32_t r = lane; r < cnt; r += 64u)
                a.masks[(int64_t)(NNB - 1 - k) * P.n + s + r] = 0ull;
        }
    }
};

// SPH density, the energy update and the masks of one cell per wave (SPLIT: per
// workgroup).
template <class M, bool LUCY, bool SPLIT>
__device__ __forceinline__ void density_cells(const DensityArgs &a, uint32_t blk,
                                              DensityLds<M, SPLIT> &lds)
{
    const DevParams &P = a.P;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr uint32_t kCells = SPLIT ? 1u : (uint32_t)kCellWaves;
    const uint32_t c0 = blk * kCells, c = SPLIT ? c0 : c0 + (uint32_t)w;
    const uint32_t g0 = a.cell_start[c0];
    const uint32_t g1 = a.cell_start[min((int64_t)c0 + kCells, P.ncell)];
    const bool tail = g1 - g0 <= (uint32_t)kTail;
    if (c < P.ncell) {
        const CellWave cw(P, CellXyz(P, c), a.cell_start);
        const int m = (int)cw.m, q = SPLIT ? (m + kCellWaves - 1) / kCellWaves : m;
        const int lo = SPLIT ? min(w * q, m) : 0, hi = SPLIT ? min(lo + q, m) : m;
        DensityWave<M, LUCY, SPLIT> d{a, P, cw, lds, lane, w, lo, hi};
        d.run();
        if (tail) {   // (an overflowing cell keeps its densities)
            if (cw.m == 0u)
                for (uint32_t r = lane; r < lane_of(cw.raw, OWN_NB); r += 64u)
                    lds.rho[cw.own - g0 + r] = -1.0;
            else if (lane >= lo && lane < hi)
                lds.rho[cw.own - g0 + (uint32_t)lane] = M::density_scale(P, d.acc);
        } else if (lane >= lo && lane < hi) {
            density_store(a, cw.own + lane, M::density_scale(P, d.acc));
        }
    }
    if (!tail) return;
    // the workgroup's particles are consecutive: the energy update (a power per
    // particle) at full lane occupancy
    __syncthreads();
    if (threadIdx.x < g1 - g0) {
        const double rho = lds.rho[threadIdx.x];
        if (!(rho < 0.0)) density_store(a, g0 + threadIdx.x, rho);
    }
}

// ---------------------------------------------------------------- forces
struct ForcesArgs {
    DevParams P;
    const void *q4;          // packed records of the model: x, y, z, Pi
    const uint32_t *cell_sorted, *cell_start;
    const uint64_t *masks;
    double *f, *p;
    int half_kick;
};

__device__ __forceinline__ void force_store(const ForcesArgs &a, int64_t i, int axis, double f)
{
    const int64_t at = axis * a.P.n + i;
    a.f[at] = f;
    if (a.half_kick) a.p[at] += 0.5 * a.P.dt * f;
}

// One lane per particle: one loop over the lane's partners in the fixed order.
// The trip count is the lane's partner count, and a lane moves on to its next
// non-empty neighbour cell inside the loop body, whose cell start and mask are
// loaded one cell ahead.  A wave then runs as many iterations as its busiest
// lane has partners, instead of the sum over the cells of the busiest lane in
// each.  EDGE: some lane of the wave sits in a first or last cell of an axis,
// where neighbour steps wrap and carry a periodic shift; elsewhere cell k is
// c + o_x + o_y n_x + o_z n_x n_y - (1 + n_x + n_x n_y) for the offset digits o
// of k.
template <class M, bool LUCY, bool EDGE>
__device__ __forceinline__ void forces_lane_loop(const ForcesArgs &a, int64_t i, uint32_t c,
                                                 const NbSteps &nb, uint32_t todo, int total,
                                                 typename M::Vec qi, typename M::Real f[3])
{
    typedef typename M::Real Real;
    const DevParams &P = a.P;
    const Real *__restrict__ q4 = static_cast<const Real *>(a.q4);
    const int64_t n = P.n;
    const uint32_t nx = (uint32_t)P.nc[0], nxy = nx * (uint32_t)P.nc[1];
    const uint32_t c0 = c - 1u - nx - nxy;
    constexpr bool SHIFT = EDGE || M::kShiftEverywhere;
    const Real ms = M::force_scale(P);
    struct Cell {
        uint32_t start;
        uint64_t mask;
        Real sh[3];
    };
    auto cell = [&](int k) {   // start and mask requested, shift set
        Cell r;
        const uint32_t q3 = ((uint32_t)k * 11u) >> 5;   // k / 3 for k < 27
        const uint32_t o[3] = {(uint32_t)k - 3u * q3, q3 - 3u * ((q3 * 11u) >> 5),
                               (q3 * 11u) >> 5};
        uint32_t cn = c0 + o[0] + o[1] * nx + o[2] * nxy;
        if (EDGE) cn = (uint32_t)nb.get(P, k).c;
        if (SHIFT)
            for (int x = 0; x < 3; ++x)
                r.sh[x] = M::shift(P, x, (int)o[x], (nb.lo >> x) & 1u, (nb.hi >> x) & 1u);
        r.start = a.cell_start[cn];
        r.mask = a.masks[(int64_t)k * n + i];
        return r;
    };
    Cell cur, next;
    cur.mask = next.mask = 0ull;
    cur.start = next.start = 0u;
    for (int x = 0; x < 3; ++x) cur.sh[x] = next.sh[x] = (Real)0;
    if (todo) {
        next = cell(__builtin_ctz(todo));
        todo &= todo - 1u;
    }
    for (int t = 0; t < total; ++t) {
        if (cur.mask == 0ull) {   // the prefetched cell becomes current
            cur = next;
            if (todo) {
                next = cell(__builtin_ctz(todo));
                todo &= todo - 1u;
            }
        }
        const uint32_t j = cur.start + (uint32_t)__builtin_ctzll(cur.mask);
        cur.mask &= cur.mask - 1ull;
        const typename M::Vec qj = load_vec<M>(q4, j);
        Real dx = qi.x - qj.x, dy = qi.y - qj.y, dz = qi.z - qj.z;
        if (SHIFT) {
            dx += cur.sh[0];
            dy += cur.sh[1];
            dz += cur.sh[2];
        }
        const Real r2 = dx * dx + dy * dy + dz * dz;
        const Real sc = ms * (qi.w + qj.w) * M::template force<LUCY>(P, r2);
        f[0] += sc * dx;
        f[1] += sc * dy;
        f[2] += sc * dz;
    }
}

// G = 3: one loop per layer of nine neighbour cells (offsets 9l .. 9l + 8,
// equal z offset), so that the lanes of a wave read the records of nearby
// cells at about the same time; G = 1: one loop over all 27 (the same sums in
// the same order either way)
template <class M, bool LUCY, int G>
__device__ __forceinline__ void forces_lane(const ForcesArgs &a, uint32_t blk)
{
    const DevParams &P = a.P;
    const int64_t i = (int64_t)blk * blockDim.x + threadIdx.x;
    if (i >= P.n) return;
    const uint32_t c = a.cell_sorted[i];
    const CellXyz cc(P, c);
    const NbSteps nb(P, cc.x, cc.y, cc.z);
    const typename M::Vec qi = load_vec<M>(static_cast<const typename M::Real *>(a.q4), i);
    const bool edge = __any((nb.lo | nb.hi) != 0u);
    typename M::Real f[3] = {0, 0, 0};
    for (int g = 0; g < G; ++g) {
        // non-empty neighbour cells (bit k) and the number of partners
        uint32_t todo = 0u;
        int total = 0;
        for (int k = g * (27 / G); k < (g + 1) * (27 / G); ++k) {
            const uint64_t m = a.masks[(int64_t)k * P.n + i];
            todo |= (m != 0ull ? 1u : 0u) << k;
            total += __popcll(m);
        }
        if (edge) forces_lane_loop<M, LUCY, true>(a, i, c, nb, todo, total, qi, f);
        else forces_lane_loop<M, LUCY, false>(a, i, c, nb, todo, total, qi, f);
    }
    for (int x = 0; x < 3; ++x) force_store(a, i, x, (double)f[x]);
}

// sum of v[0 .. count) in order, added to acc; eight values in flight (zeros
// behind the last one)
template <class Real>
__device__ __forceinline__ Real ordered_sum(const Real *v, int count, Real acc)
{
    for (int r = 0; r < count; r += 8) {
        Real x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = v[r + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = acc + x[u];
    }
    return acc;
}

// The partners of particle i, 256 at a time, into LDS entries j | k << 27 in
// the fixed order (lane k expands the mask of neighbour cell k from its place
// on); one wave per particle, boxes below 2^27 particles.
struct WavePartners {
    static constexpr int kWindow = 256;
    uint64_t mask;       // lane k: partners in cell k not yet written
    uint32_t start;      // lane k: first particle of cell k
    int at, total;       // lane k: place of its next partner; all partners

    __device__ __forceinline__ WavePartners(const DevParams &P, const NbSteps &nb,
                                            const uint32_t *cell_start, const uint64_t *masks,
                                            int64_t i)
    {
        const int lane = threadIdx.x & 63;
        mask = 0ull;
        start = 0u;
        if (lane < NNB) {
            start = cell_start[nb.get(P, lane).c];
            mask = masks[(int64_t)lane * P.n + i];
        }
        int incl = __popcll(mask);
        at = -incl;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        at += incl;
        total = __builtin_amdgcn_readlane(incl, NNB - 1);
    }
    __device__ __forceinline__ void window(uint32_t *ent, int w0)
    {
        const int limit = w0 + kWindow;
        while (__any(mask != 0ull && at < limit))
            if (mask != 0ull && at < limit) {
                ent[at - w0] = (start + (uint32_t)__builtin_ctzll(mask)) |
                               ((threadIdx.x & 63u) << 27);
                mask &= mask - 1ull;
                ++at;
            }
        wave_sync();
    }
};

// separation q_i - q_j of entry e (see WavePartners)
template <class M>
__device__ __forceinline__ void partner_separation(const DevParams &P, const NbSteps &nb,
                                                   uint32_t e, const typename M::Vec &qi,
                                                   const typename M::Vec &qj,
                                                   typename M::Real d[3])
{
    d[0] = qi.x - qj.x;
    d[1] = qi.y - qj.y;
    d[2] = qi.z - qj.z;
    if (M::kShiftEverywhere || (nb.lo | nb.hi) != 0u) {
        const int k = (int)(e >> 27), o[3] = {k % 3, (k / 3) % 3, k / 9};
        for (int x = 0; x < 3; ++x)
            d[x] += M::shift(P, x, o[x], (nb.lo >> x) & 1u, (nb.hi >> x) & 1u);
    }
}

// One wave per particle: 64 partners at a time, their terms into LDS, added up
// in order by one lane per component.
template <class M, bool LUCY>
__device__ __forceinline__ void forces_wave(const ForcesArgs &a, int64_t i, uint32_t *ent,
                                            typename M::Real (*terms)[64])
{
    typedef typename M::Real Real;
    const DevParams &P = a.P;
    const int lane = threadIdx.x & 63;
    const Real *q4 = static_cast<const Real *>(a.q4);
    const CellXyz cc(P, (uint32_t)__builtin_amdgcn_readfirstlane((int)a.cell_sorted[i]));
    const NbSteps nb(P, cc.x, cc.y, cc.z);
    const typename M::Vec qi = load_vec<M>(q4, i);
    WavePartners partners(P, nb, a.cell_start, a.masks, i);
    const Real ms = M::force_scale(P);
    Real f = (Real)0;        // lane x < 3: component x
    for (int w0 = 0; w0 < partners.total; w0 += WavePartners::kWindow) {
        partners.window(ent, w0);
        const int cnt = min(partners.total - w0, WavePartners::kWindow);
        for (int t0 = 0; t0 < cnt; t0 += 64) {
            Real v[3] = {0, 0, 0};
            if (t0 + lane < cnt) {
                const uint32_t e = ent[t0 + lane];
                const typename M::Vec qj = load_vec<M>(q4, e & ((1u << 27) - 1u));
                Real d[3];
                partner_separation<M>(P, nb, e, qi, qj, d);
                const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                const Real sc = ms * (qi.w + qj.w) * M::template force<LUCY>(P, r2);
                for (int x = 0; x < 3; ++x) v[x] = sc * d[x];
            }
            for (int x = 0; x < 3; ++x) terms[x][lane] = v[x];
            wave_sync();
            if (lane < 3) f = ordered_sum(terms[lane], min(cnt - t0, 64), f);
            wave_sync();
        }
    }
    if (lane < 3) force_store(a, i, lane, (double)f);
}

// ---------------------------------------------------------------- launches
// Both passes choose their form by the box; in launches recorded for a batch all
// boxes share the GPU, and take the forms of large ones.  The forms agree bit for
// bit.
// Density: four waves per cell up to 2^10 cells, one per SIMD of the GPU (384
// cells: 25 us against 50; 1728 cells: 53 against 54; 7128: 102 against 73).
constexpr int64_t kSplitMaxCells = 1 << 10;
// Forces: a wave per particle up to 48k particles (1000: 13 us against 56, 8064:
// 20 against 59, 31680: 42 against 64, 100003: 96 against 70).
constexpr int64_t kWaveMaxParticles = 48 << 10;

template <class M, bool LUCY>
__device__ __forceinline__ void density_body(const DensityArgs &a, uint32_t blk)
{
    __shared__ DensityLds<M, false> lds;
    density_cells<M, LUCY, false>(a, blk, lds);
}
template <class M, bool LUCY, bool SPLIT>
__global__ __launch_bounds__(64 * kCellWaves) void k_density(DensityArgs a)
{
    __shared__ DensityLds<M, SPLIT> lds;
    density_cells<M, LUCY, SPLIT>(a, xcd_block(blockIdx.x, gridDim.x), lds);
}
template <class M, bool LUCY, int G>
__global__ __launch_bounds__(256) void k_forces(ForcesArgs a)
{
    forces_lane<M, LUCY, G>(a, xcd_block(blockIdx.x, gridDim.x));
}
template <class M, bool LUCY>
__global__ __launch_bounds__(256) void k_forces_wave(ForcesArgs a)
{
    __shared__ uint32_t ent[4][WavePartners::kWindow];
    __shared__ typename M::Real terms[4][3][64];
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t i = 4 * (int64_t)blockIdx.x + w;
    if (i < a.P.n) forces_wave<M, LUCY>(a, i, ent[w], terms[w]);
}

// (multi: the multi-box forms of this model and kernel)
template <class M, bool LUCY>
int launch_density(sdpd_ctx *c, const DensityArgs &args, MultiKernel multi)
{
    if (c->ncell <= kSplitMaxCells && !c->rec) {
        hipLaunchKernelGGL((k_density<M, LUCY, true>), dim3((unsigned)c->ncell),
                           dim3(64 * kCellWaves), 0, c->stream, args);
        return check_hip(hipGetLastError());
    }
    return launch_or_record(c, k_density<M, LUCY, false>, multi,
                            (unsigned)((c->ncell + kCellWaves - 1) / kCellWaves),
                            64 * kCellWaves, 0, args);
}
template <class M, bool LUCY>
int launch_forces(sdpd_ctx *c, const ForcesArgs &args, MultiKernel multi)
{
    if (c->n <= kWaveMaxParticles && !c->rec) {
        hipLaunchKernelGGL((k_forces_wave<M, LUCY>), dim3((unsigned)((c->n + 3) / 4)), dim3(256),
                           0, c->stream, args);
        return check_hip(hipGetLastError());
    }
    return launch_or_record(c, k_forces<M, LUCY, 3>, multi, (unsigned)((c->n + 255) / 256), 256,
                            0, args);
}

}  // namespace sdpd
