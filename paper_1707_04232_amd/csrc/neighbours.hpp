// Loops over the neighbour candidates and partners of a particle, shared by
// the FP64 and the FP32 (mixed precision) particle passes.
#pragma once

#include "sdpd_internal.hpp"
#include "fd_elem.hpp"

#include <float.h>

#include <algorithm>
#include <type_traits>

namespace sdpd {

// ---------------------------------------------------------------- arithmetic
// A model of the arithmetic: the type of positions and sums, the packed record
// (x, y, z and a scalar), the periodic shift of axis a for neighbour offset o
// (0, 1, 2) of a cell that is the first (lo) or the last (hi) of the axis, the
// active test and the terms.  Densities are summed in candidate order (offset
// index k = 0..26 with z slowest, then slot).

// FP64: absolute positions; the image is chosen per neighbour cell: a cell
// reached across the box boundary contributes (x_i - x_j) +- L, which is the
// minimum-image difference for every pair closer than h (L >= 4 h), in the
// same rounding as the plain form.
struct ModelF64 {
    typedef double Real;
    typedef double4 Vec;
    static constexpr bool kShiftEverywhere = false;
    static constexpr int kDensityOcc = 5;
    static constexpr int kChunks = 3;                    // see DensityWave
    static constexpr int kLanes = 8;                     // see PartnerSums
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
    static constexpr int kDensityOcc = 7;
    static constexpr int kChunks = 3;
    static constexpr int kLanes = 4;
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

// x of another lane (CTRL: the DPP control word)
template <int CTRL>
__device__ __forceinline__ float moved(float x)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double moved(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

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
    // the cell of position t < total and the particle there; called by the whole
    // wave (a lane that is switched off gives no value to the others)
    __device__ __forceinline__ void find(uint32_t t, int &k, uint32_t &j) const
    {
        k = 0;
#pragma unroll
        for (int step = 16; step; step >>= 1)
            if ((uint32_t)__shfl((int)b, k + step) <= t) k += step;
        j = (uint32_t)__shfl((int)s, k) + (t - (uint32_t)__shfl((int)b, k));
    }
};

// ---------------------------------------------------------------- density
struct DensityArgs {
    DevParams P;
    const void *q4;          // packed records of the model
    const uint32_t *cell_sorted, *cell_start;
    double *rho, *eps;
    int update_eps;
    uint64_t *masks;         // masks[(k - 13) n + i]: slot bits of the partners in cell k,
                             // k = 13 (the own cell, without i itself) .. 26
    // partners of particle i (itself included) in candidate order: entry r < list_len at
    // list[list_len i + r], the others behind these parts of all particles, at
    // list[list_len n + (list_cap - list_len) i + r - list_len]; r < count[i]; complete
    // if count <= list_cap
    uint32_t *list, *count;
    uint32_t list_len, list_cap;
    uint32_t *err;
    double *rho_w;           // FP64: also into the w slot of the record, or NULL
    float reach2;            // h^2 and the rounding of the FP32 test for it (density_reach2)
    const uint32_t *dense;   // not zero: a cell holds kDenseRegion particles or more
};

// Squared distance, in FP32, up to which a candidate is kept for the tests: the
// separations are rounded relative to positions of up to two cell edges (2^-24 of
// them, three times per axis), which moves the square by less than 2.2e-6 h edge
// (h^2 is a relative 1e-4 of its own apart; cells may be much wider than h).
inline float density_reach2(const DevParams &P)
{
    double edge = 0.0;
    for (int a = 0; a < 3; ++a) edge = std::max(edge, 1.0 / P.inv_cell[a]);
    return (float)(P.h * P.h * 1.0001 + 8e-6 * P.h * edge + 1e-11 * edge * edge);
}

// an entry of the list: particle and offset index
__device__ __forceinline__ uint32_t list_entry(uint32_t j, int k)
{
    return j | (uint32_t)k << kEntryBits;
}
__device__ __forceinline__ uint32_t entry_particle(uint32_t e)
{
    return e & ((1u << kEntryBits) - 1u);
}

// entry r < list_cap of particle i's list
__device__ __forceinline__ uint32_t *list_at(const DensityArgs &a, uint32_t i, uint32_t r)
{
    const int64_t at = r < a.list_len ? (int64_t)i * a.list_len + r
                                      : a.P.n * a.list_len +
                                            (int64_t)i * (a.list_cap - a.list_len) +
                                            (r - a.list_len);
    return a.list + at;
}

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

// Density, masks and partner lists, one cell per wave.  The candidates that come
// within h of the box around the cell's particles are listed in LDS, in candidate
// order, and taken into the lanes' registers 64 K at a time (a window); the wave goes
// through the cell's particles, tests its candidates against one of them at once,
// queues the squared distances in range in LDS and evaluates the kernel for the queue
// at full lane occupancy; lane i then adds up the terms of particle i in order.  The
// test of particle i is bit i of a lane's word, which ends as the mask of its
// candidate for this cell: no pair is looked at twice and no mask is taken apart.
//
// Bound by the VALU: of 460 candidates per particle (17 per cell, h = 0.98 cell
// edges) 310 are in reach of the cell, 4.8 lane-parallel tests of 16 instructions,
// and each window costs some 35 more per particle.  A thread per particle reads 24 B
// of every candidate through the L1 instead and runs to the largest cell of its wave:
// 677 us for 1M particles in FP64 (now 542, of which the list takes 120), 251 us for
// 262k (156), 168 us for 137k in FP32 (84), 3590 us for 8M (3310).  Without the test
// against the box: 601, 195, 88, 3400.
//
// The list saves the force and gradient passes the walk through the masks (1M
// particles: forces 410 -> 216 us).  A window's entries of a particle go through
// LDS and out in one store; storing them where they are found took 8 % longer, and a
// queue of entries beside that of the terms, emptied with it, 12 %.
//
// K: more candidates per lane mean fewer windows and fewer waves per SIMD.  1M
// particles, K = 2, 3, 4, 5: 543, 542, 578, 615 us; 8M in FP32, K = 2, 3, 4, 5: 3362,
// 3313, 3658, 3615.  kDensityOcc: the waves per SIMD that the compiler has to allow
// (1M particles, 4 and 5: 8 % apart).
constexpr int kTerms = 576;        // queue entries of a wave
constexpr int kTail = 256;         // particles of a workgroup's shared last part

// WAVES: those of the workgroup
template <class M, bool SPLIT, int WAVES = kCellWaves>
struct DensityLds {
    typename M::Real terms[WAVES][kTerms + 64];
    double rho[WAVES > 1 ? kTail : 1];
    uint32_t near[WAVES][64 * M::kChunks + 64];   // candidates that are not out of reach
    uint32_t part[WAVES][64 * M::kChunks + 64];   // list entries of a particle and window
    uint32_t words[SPLIT ? WAVES : 1][SPLIT ? 64 * WAVES : 1];
};

// SPLIT: the workgroup's waves share one cell, wave w with the particles in
// slots w q .. w q + q - 1 (q = ceil(m / 4)) of it, and put their words together
// in LDS: for boxes of so few cells that a wave per cell leaves SIMDs idle and the
// pass takes as long as one wave's chain (1000 particles: 18 us, a wave per cell
// 34, four lanes of a thread per particle 66)
template <class M, bool LUCY, bool SPLIT, int WAVES = kCellWaves>
struct DensityWave {
    typedef typename M::Real Real;
    const DensityArgs &a;
    const DevParams &P;
    const CellWave &cw;
    DensityLds<M, SPLIT, WAVES> &lds;
    const int lane, wave, lo, hi;   // slots lo .. hi - 1 are this wave's
    Real *terms;
    Real x, y, z, acc;       // lane i < m: particle i of the cell and its sum
    Real x0[3];              // particle 0
    float box_lo[3], box_hi[3];   // the box around the cell's particles, relative to it
    uint32_t beg, end;       // ... its terms in the queue
    uint32_t partners;       // ... its list entries
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

    // WORDS: the window has cells whose masks for this one are kept
    template <bool SHIFT, int K, bool WORDS>
    __device__ __forceinline__ void window(uint32_t width)
    {
        const Real *__restrict__ q4 = static_cast<const Real *>(a.q4);
        const int chunks = (int)((width + 63u) / 64u);
        Real cx[K], cy[K], cz[K], sh[K][3];
        uint32_t entry[K];
#pragma unroll
        for (int c = 0; c < K; ++c) {
            cx[c] = cy[c] = cz[c] = (Real)0;
            entry[c] = 0u;
            for (int d = 0; d < 3; ++d) sh[c][d] = (Real)0;
            if (c >= chunks) continue;
            const uint32_t t = 64u * c + lane;
            const uint32_t e = lds.near[wave][min(t, width - 1u)];
            const uint32_t j = entry_particle(e);
            const int k = (int)(e >> kEntryBits);
            const typename M::Vec v = load_vec<M>(q4, j);
            // a lane past the end: out of range of everything
            cx[c] = t < width ? v.x : (Real)1e18;
            cy[c] = v.y;
            cz[c] = v.z;
            entry[c] = e;
            if (SHIFT) {
                const int o[3] = {k % 3, (k / 3) % 3, k / 9};
                for (int d = 0; d < 3; ++d)
                    sh[c][d] = M::shift(P, d, o[d], (cw.steps.lo >> d) & 1u,
                                        (cw.steps.hi >> d) & 1u);
            }
        }
        const int m = (int)cw.m;
        constexpr bool kHalf = WAVES == 1;   // lo .. hi - 1 within a word of the masks
        const int last_half = kHalf ? lo >> 5 : 0;
        for (int half = (kHalf ? hi : m) > 32 ? 1 : 0; half >= last_half; --half) {
            uint32_t w[K];
#pragma unroll
            for (int c = 0; c < K; ++c) w[c] = 0u;
            const int first_slot = max(lo, 32 * half);
            for (int i = min(hi, 32 * half + 32) - 1; i >= first_slot; --i) {
                const Real xi = lane_of(x, i), yi = lane_of(y, i), zi = lane_of(z, i);
                if (fill + 64u * K + 3u > (uint32_t)kTerms) flush();
                const uint32_t first = fill, had = lane_of(partners, i);
                uint32_t total = 0u;
                uint32_t *const list = a.list + (int64_t)(cw.own + (uint32_t)i) * a.list_len;
                Real *const unused = terms + kTerms + lane;
                uint32_t *const part = lds.part[wave], *const unused_part = part + 64 * K + lane;
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
                    if (WORDS) w[c] = w[c] + w[c] + (near ? 1u : 0u);
                    // (no branch: the other lanes write to slots that nothing reads)
                    uint32_t at = below(hit, 0u);
                    asm volatile("" : "+v"(at));   // (computed, not branched around)
                    *(near ? terms + fill + at : unused) = r2;
                    *(near ? part + total + at : unused_part) = entry[c];
                    fill += (uint32_t)__popcll(hit);
                    total += (uint32_t)__popcll(hit);
                }
                // the window's part of the list
                wave_sync();
                if (had + total <= a.list_len)
                    for (uint32_t r = lane; r < total; r += 64u) list[had + r] = part[r];
                else if (had + total <= a.list_cap)
                    for (uint32_t r = lane; r < total; r += 64u)
                        *list_at(a, cw.own + (uint32_t)i, had + r) = part[r];
                wave_sync();
                // up to a multiple of four with entries without a term
                if (lane < 3) terms[fill + lane] = (Real)-1;
                fill = (fill + 3u) & ~3u;
                if (lane == i) {
                    beg = first;
                    end = fill;
                    partners = had + total;
                }
            }
            if (!WORDS) continue;
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
                    const uint32_t k = entry[c] >> kEntryBits, j = entry_particle(entry[c]);
                    if (k > (uint32_t)OWN_NB) continue;
                    uint32_t v = w[c];
                    if (SPLIT) {
                        v = 0u;
                        for (int o = 0; o < kCellWaves; ++o) v |= lds.words[o][64 * c + lane];
                    }
                    // i itself is no partner
                    const uint32_t slot = j - cw.own;
                    if (k == (uint32_t)OWN_NB && (slot >> 5) == (uint32_t)half)
                        v &= ~(1u << (slot & 31u));
                    const int64_t e = (int64_t)((uint32_t)OWN_NB - k) * P.n + j;
                    if (m > 32) words[2 * e + half] = v;
                    else a.masks[e] = v;
                }
            }
        }
    }

    template <bool SHIFT, int K>
    __device__ __forceinline__ void windows()
    {
        uint32_t *const near = lds.near[wave];
        uint32_t held = 0u;
        for (uint32_t pos = 0u; pos < cw.total || held;) {
            for (; held < 64u * K && pos < cw.total; pos += 64u) held = reach<SHIFT>(pos, held);
            wave_sync();
            if (held == 0u) break;
            const uint32_t width = min(held, 64u * K);
            const int k0 = __builtin_amdgcn_readfirstlane((int)(near[0] >> kEntryBits));
            if (k0 <= OWN_NB) window<SHIFT, K, true>(width);
            else window<SHIFT, K, false>(width);
            flush();   // (a lane has one segment of the queue at a time)
            const uint32_t rest = near[64 * K + lane];   // fewer than 64
            wave_sync();
            held -= width;
            if ((uint32_t)lane < held) near[lane] = rest;
        }
    }

    // Candidates pos .. pos + 63 that come within h of the box around the cell's
    // particles, behind the first `held` of the list; the masks of the others (a
    // quarter to a third of all: cells reached across a corner or an edge) are zero.
    template <bool SHIFT>
    __device__ __forceinline__ uint32_t reach(uint32_t pos, uint32_t held)
    {
        int k;
        uint32_t j;
        cw.find(min(pos + (uint32_t)lane, cw.total - 1u), k, j);   // (every lane takes part)
        const typename M::Vec v = load_vec<M>(static_cast<const Real *>(a.q4), j);
        Real d[3] = {v.x - x0[0], v.y - x0[1], v.z - x0[2]};
        if (SHIFT) {
            const int o[3] = {k % 3, (k / 3) % 3, k / 9};
            for (int c = 0; c < 3; ++c)
                d[c] -= M::shift(P, c, o[c], (cw.steps.lo >> c) & 1u, (cw.steps.hi >> c) & 1u);
        }
        float r2 = 0.0f;
        for (int c = 0; c < 3; ++c) {
            const float g = (float)d[c], t = fmaxf(fmaxf(box_lo[c] - g, g - box_hi[c]), 0.0f);
            r2 += t * t;
        }
        const bool in = pos + (uint32_t)lane < cw.total, keep = in && r2 <= a.reach2;
        const uint64_t kept = __ballot(keep);
        if (keep) lds.near[wave][held + below(kept, 0u)] = list_entry(j, k);
        else if (in && k <= OWN_NB) a.masks[(int64_t)(OWN_NB - k) * P.n + j] = 0ull;
        return held + (uint32_t)__popcll(kept);
    }

    // smallest value of the wave (rows of 16 lanes, then the four rows)
    static __device__ __forceinline__ float wave_min(float v)
    {
        v = fminf(v, moved<0xb1>(v));
        v = fminf(v, moved<0x4e>(v));
        v = fminf(v, moved<0x141>(v));
        v = fminf(v, moved<0x140>(v));
        return fminf(fminf(lane_of(v, 0), lane_of(v, 16)), fminf(lane_of(v, 32), lane_of(v, 48)));
    }

    __device__ __forceinline__ void run()
    {
        terms = lds.terms[wave];
        x = y = z = acc = (Real)0;
        beg = end = fill = partners = 0u;
        if ((uint32_t)lane < cw.m) {
            const typename M::Vec v =
                load_vec<M>(static_cast<const Real *>(a.q4), cw.own + (uint32_t)lane);
            x = v.x;
            y = v.y;
            z = v.z;
        }
        x0[0] = lane_of(x, 0);
        x0[1] = lane_of(y, 0);
        x0[2] = lane_of(z, 0);
        const float rel[3] = {(float)(x - x0[0]), (float)(y - x0[1]), (float)(z - x0[2])};
        for (int c = 0; c < 3; ++c) {   // (empty cell: nothing is in reach)
            const bool own = (uint32_t)lane < cw.m;
            box_lo[c] = wave_min(own ? rel[c] : FLT_MAX);
            box_hi[c] = -wave_min(own ? -rel[c] : FLT_MAX);
        }
        if (M::kShiftEverywhere || cw.edge()) windows<true, M::kChunks>();
        else windows<false, M::kChunks>();
        // overflowing cells: reported, not visited
        uint64_t over = __ballot(cw.raw != cw.cnt);
        if (over && lane == 0) atomicOr(a.err, ERR_CELLCAP);
        for (; over; over &= over - 1ull) {
            const int k = __builtin_ctzll(over);
            if (k > OWN_NB) break;
            const uint32_t s = lane_of(cw.s, k), cnt = lane_of(cw.raw, k);
            for (uint32_t r = lane; r < cnt; r += 64u) {
                a.masks[(int64_t)(OWN_NB - k) * P.n + s + r] = 0ull;
                if (k == OWN_NB) a.count[s + r] = 0u;
            }
        }
        if (lane >= lo && lane < hi) a.count[cw.own + (uint32_t)lane] = partners;
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

// The same sums, masks and lists, bit for bit (where no cell overflows), for large boxes
// whose cells are mostly empty or hold few particles: a wave per cell then mostly finds
// that there is nothing to do.  A lane per particle (density_lanes), but where the cell
// pass has found cells of kDenseRegion particles for the cells of dense regions, those with
// kDenseCell particles and more and the cells around them: they are taken by a wave each
// (density_dense), the wave that has the cell's first particle among its kHeads ones, and
// cells of more than 32 particles by two, one for each word of their masks.  One wave per
// workgroup: most find one such cell or none, and a workgroup's LDS is held until its last
// wave is done.
//
// us, lanes only and now: a droplet of 10^5 particles at h = 2.5 spacings in 60^3 cells
// 184, 137, at h = 3.6 in 40^3 452, 262 (a wave for all of a cell 362), one of 10^6 at h =
// 3.4 in 88^3 cells 1673, 1069, in FP32 1434, 839; uniform boxes of one and three particles
// per cell 48, 53 and 91, 98 (the launch that finds no dense cell; with both in one launch,
// lanes in workgroups of one wave too, 55 and 107).
constexpr uint32_t kDenseCell = 10u;
constexpr int kHeads = 16;

// The dense cells whose slot 0 or 32 is among particles kHeads blk .. kHeads blk + kHeads - 1
template <class M, bool LUCY>
__device__ __forceinline__ void density_dense(const DensityArgs &a, uint32_t blk)
{
    __shared__ DensityLds<M, false, 1> lds;
    if (*a.dense == 0u) return;
    const DevParams &P = a.P;
    const int lane = threadIdx.x;
    const int64_t i = (int64_t)blk * kHeads + lane;
    uint32_t c = 0u;
    bool dense = false;
    if (lane < kHeads && i < P.n) {
        c = a.cell_sorted[i];
        if (((i - (int64_t)a.cell_start[c]) & 31) == 0) {
            const CellXyz cc(P, c);
            const NbSteps steps(P, cc.x, cc.y, cc.z);
#pragma unroll
            for (int k = 0; k < NNB; ++k) {
                const uint32_t cn = (uint32_t)steps.get(P, k).c;
                dense = dense || a.cell_start[cn + 1] - a.cell_start[cn] >= kDenseCell;
            }
        }
    }
    for (uint64_t heads = __ballot(dense); heads; heads &= heads - 1ull) {
        const DensityArgs &b = reread(a);   // (not held through the loop)
        const int l = __builtin_ctzll(heads);
        const CellXyz cc(b.P, lane_of(c, l));
        const CellWave cw(b.P, cc, b.cell_start);
        // slots 0 .. 31 or 32 .. 63; all of an overflowing cell's particles are done once
        const int m = (int)cw.m, lo = (int)((uint32_t)blk * kHeads + (uint32_t)l - cw.own);
        if (lo > 0 && lo >= m) continue;
        DensityWave<M, LUCY, false, 1> d{b, b.P, cw, lds, lane, 0, lo, min(lo + 32, m)};
        d.run();
        if (lane >= d.lo && lane < d.hi)
            density_store(b, cw.own + lane, M::density_scale(b.P, d.acc));
    }
}

// The particles of the other cells, and of all particles the masks for the cells ahead
// that no wave takes (a wave writes those for its cell).  DENSE: there are dense cells.
template <class M, bool LUCY, bool DENSE>
__device__ __forceinline__ void density_lanes(const DensityArgs &a, uint32_t blk)
{
    typedef typename M::Real Real;
    const DevParams &P = a.P;
    const int64_t n = P.n, i = (int64_t)blk * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const Real *__restrict__ q4 = static_cast<const Real *>(a.q4);
    const uint32_t c = a.cell_sorted[i];
    const CellXyz cc(P, c);
    const NbSteps steps(P, cc.x, cc.y, cc.z);
    if (DENSE && a.cell_start[c + 1] - a.cell_start[c] >= kDenseCell) {
        // a wave takes all cells around it but empty ones
#pragma unroll
        for (int k = OWN_NB + 1; k < NNB; ++k) {
            const uint32_t cn = (uint32_t)steps.get(P, k).c;
            if (a.cell_start[cn + 1] == a.cell_start[cn])
                a.masks[(int64_t)(k - OWN_NB) * n + i] = 0ull;
        }
        return;
    }
    bool dense = false;   // a wave takes this particle's cell: only masks are left to do
    if (DENSE) {
#pragma unroll
        for (int k = 0; k < NNB; ++k) {
            const uint32_t cn = (uint32_t)steps.get(P, k).c;
            dense = dense || a.cell_start[cn + 1] - a.cell_start[cn] >= kDenseCell;
        }
    }
    const typename M::Vec qi = load_vec<M>(q4, i);
    Real acc = (Real)0;
    uint32_t partners = 0u;
    for (int k = dense ? OWN_NB : 0; k < NNB; ++k) {
        const int o[3] = {k % 3, (k / 3) % 3, k / 9};
        const uint32_t cn = (uint32_t)steps.get(P, k).c, s = a.cell_start[cn];
        uint32_t cnt = a.cell_start[cn + 1] - s;
        if (DENSE && cnt >= kDenseCell) continue;
        if (cnt > (uint32_t)P.cap) {   // overflowing cell: reported, not visited
            atomicOr(a.err, ERR_CELLCAP);
            cnt = 0u;
        }
        Real sh[3];
        for (int x = 0; x < 3; ++x)
            sh[x] = M::shift(P, x, o[x], (steps.lo >> x) & 1u, (steps.hi >> x) & 1u);
        uint64_t mask = 0ull;
        for (uint32_t t = 0; t < cnt; ++t) {
            const typename M::Vec v = load_vec<M>(q4, s + t);
            const Real dx = (qi.x - v.x) + sh[0], dy = (qi.y - v.y) + sh[1],
                       dz = (qi.z - v.z) + sh[2];
            const Real r2 = dx * dx + dy * dy + dz * dz;
            if (!M::near(P, r2)) continue;
            mask |= 1ull << t;
            if (DENSE && dense) continue;
            acc = acc + M::template density<LUCY>(P, r2);
            if (partners < a.list_cap)
                *list_at(a, (uint32_t)i, partners) = list_entry(s + t, k);
            ++partners;
        }
        if (k == OWN_NB && cnt) mask &= ~(1ull << (i - (int64_t)s));   // i itself is no partner
        if (k >= OWN_NB) a.masks[(int64_t)(k - OWN_NB) * n + i] = mask;
    }
    if (DENSE && dense) return;
    a.count[i] = partners;
    density_store(a, i, M::density_scale(P, acc));
}

template <class M, bool LUCY>
__device__ __forceinline__ void density_sparse(const DensityArgs &a, uint32_t blk)
{
    if (*a.dense == 0u) density_lanes<M, LUCY, false>(a, blk);
    else density_lanes<M, LUCY, true>(a, blk);
}

// ---------------------------------------------------------------- partner sums
// Sums over a particle's partners, from the lists of the density pass (same
// positions): kLanes lanes per particle, lane s with entries s, s + kLanes, ...
// FP64: each lane adds up its own and the lanes are added at the end; FP32: every
// lane adds the terms of all in list order.  Particles with more partners than the
// list holds are looked up among their candidates by the whole wave.
//
// Bound by the gathers of the partners' records (two 16 B loads per pair, 22 clocks
// each in the address unit) and, in small boxes, by the chain of a lane.  A lane per
// particle that walks the 27 masks took 410 us for 1M particles (now 216), 56 for
// 1000 (13), 2170 for 8M in FP32 (1470); the gradient's two passes at 262k particles
// 580 us.  Lanes per particle: FP64 8 (4: 284 us at 1M), FP32 4 (8 with sums through
// LDS: 2570 at 8M).  Lists that begin on cache lines: 225 -> 216, 1680 -> 1470.
struct PartnerArgs {
    DevParams P;
    const void *q4;          // packed records of the model
    const uint32_t *cell_sorted, *cell_start;
    const uint32_t *list, *count;   // (see DensityArgs)
    uint32_t list_len, list_cap;
};

// Value v of the sum over particle i's partners in lane s == v < NV of its lanes.
// term(j, own, q_i, q_j, d, r2, out): the NV values of partner j at separation d = q_i -
// q_j; term.at(i): called before with the particle of the lane.  own: j is the particle
// itself, which its list holds and ends with: zero, whatever its values (they may not be
// finite).
template <class M, int NV, class Term>
struct PartnerSums {
    typedef typename M::Real Real;
    static constexpr int kLanes = M::kLanes;
    const PartnerArgs &a;
    const DevParams &P;
    float4 *shift;           // FP32: 27 entries in LDS
    const int lane;
    const uint32_t s;

    // a particle without a complete list (uniform in the wave)
    __device__ __forceinline__ void direct(int64_t i, Term term, Real sum[NV])
    {
        const CellXyz cc(P, (uint32_t)__builtin_amdgcn_readfirstlane((int)a.cell_sorted[i]));
        const CellWave cw(P, cc, a.cell_start);
        const typename M::Vec qi = load_vec<M>(static_cast<const Real *>(a.q4), i);
        term.at(i);
        for (int v = 0; v < NV; ++v) sum[v] = (Real)0;
        for (uint32_t t0 = 0; t0 < cw.total; t0 += 64u) {
            int k;
            uint32_t j;
            cw.find(min(t0 + (uint32_t)lane, cw.total - 1u), k, j);
            const typename M::Vec qj = load_vec<M>(static_cast<const Real *>(a.q4), j);
            Real d[3] = {qi.x - qj.x, qi.y - qj.y, qi.z - qj.z};
            const int o[3] = {k % 3, (k / 3) % 3, k / 9};
            for (int x = 0; x < 3; ++x)
                d[x] += M::shift(P, x, o[x], (cw.steps.lo >> x) & 1u, (cw.steps.hi >> x) & 1u);
            const Real r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
            Real out[NV];
            for (int v = 0; v < NV; ++v) out[v] = (Real)0;
            const bool hit =
                t0 + (uint32_t)lane < cw.total && M::near(P, r2) && j != (uint32_t)i;
            if (hit) term(j, false, qi, qj, d, r2, out);
            const uint64_t hits = __ballot(hit);
            for (int v = 0; v < NV; ++v) {
                if constexpr (sizeof(Real) == 8) {
                    sum[v] += out[v];
                } else {   // in candidate order (the terms of the others are zero)
                    for (uint64_t h = hits; h; h &= h - 1ull)
                        sum[v] = sum[v] + lane_of(out[v], __builtin_ctzll(h));
                }
            }
        }
        if constexpr (sizeof(Real) == 8)   // over the lanes, in each of them
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) sum[v] += __shfl_xor(sum[v], off);
    }

    __device__ __forceinline__ Real run(int64_t i, bool live, Term term)
    {
        const Real *__restrict__ q4 = static_cast<const Real *>(a.q4);
        const typename M::Vec qi = load_vec<M>(q4, i);
        const uint32_t all = live ? a.count[i] : 0u;
        const bool over = all > a.list_cap;
        // the list's two parts one after the other: the second is only there for
        // particles of dense regions, and lists of its length as well in the first
        // would lie further apart (a gradient of 262k particles took 1.4 % longer)
        const uint32_t *__restrict__ list = a.list + i * (int64_t)a.list_len;
        uint32_t left = over ? 0u : all, cnt = min(left, a.list_len);
        auto next_part = [&] {
            left -= cnt;
            if (!__any(left != 0u)) return false;
            list = a.list + P.n * a.list_len + i * (int64_t)(a.list_cap - a.list_len);
            cnt = left;
            return true;
        };
        const uint32_t self = list_entry((uint32_t)i, OWN_NB);
        term.at(i);
        Real mine = (Real)0;
        // entry r (past the end: the particle itself)
        auto entry = [&](uint32_t r) { return r < cnt ? list[r] : self; };
        if constexpr (sizeof(Real) == 8) {
            // partners across the boundary only for particles within h of it
            bool edge = false;
            const double margin = 1.001 * P.h;
            const double x[3] = {qi.x, qi.y, qi.z};
            for (int d = 0; d < 3; ++d)
                edge = edge || x[d] < margin || x[d] > P.box[d] - margin;
            double acc[NV];
            for (int v = 0; v < NV; ++v) acc[v] = 0.0;
            auto loop = [&](auto shifted) {
                constexpr bool SHIFT = decltype(shifted)::value;
                do {
                    uint32_t e[2] = {entry(s), entry(s + kLanes)};
                    for (uint32_t r = s; __any(r < cnt); r += 2 * kLanes) {
                        typename M::Vec qj[2];
                        uint32_t j[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            j[u] = entry_particle(e[u]);
                            qj[u] = load_vec<M>(q4, j[u]);
                        }
                        e[0] = entry(r + 2 * kLanes);
                        e[1] = entry(r + 3 * kLanes);
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            double d[3] = {qi.x - qj[u].x, qi.y - qj[u].y, qi.z - qj[u].z};
                            if (SHIFT)
                                for (int x = 0; x < 3; ++x)
                                    d[x] += d[x] > P.h ? -P.box[x] : (d[x] < -P.h ? P.box[x] : 0.0);
                            const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                            double out[NV];
                            term(j[u], j[u] == (uint32_t)i, qi, qj[u], d, r2, out);
                            for (int v = 0; v < NV; ++v) acc[v] += out[v];
                        }
                    }
                } while (next_part());
            };
            if (__any(edge)) loop(std::true_type());
            else loop(std::false_type());
            for (int v = 0; v < NV; ++v) {
                acc[v] += moved<0xb1>(acc[v]);    // lanes 1 0 3 2 of four
                acc[v] += moved<0x4e>(acc[v]);    // lanes 2 3 0 1
                acc[v] += moved<0x141>(acc[v]);   // eight lanes mirrored
                if (s == (uint32_t)v) mine = acc[v];
            }
        } else {
            if (lane < NNB) {
                const int o[3] = {lane % 3, (lane / 3) % 3, lane / 9};
                shift[lane] = make_float4(M::shift(P, 0, o[0], false, false),
                                          M::shift(P, 1, o[1], false, false),
                                          M::shift(P, 2, o[2], false, false), 0.0f);
            }
            wave_sync();
            float acc[NV];
            for (int v = 0; v < NV; ++v) acc[v] = 0.0f;
            do {
                uint32_t e[2] = {entry(s), entry(s + kLanes)};
                for (uint32_t r = s; __any(r < cnt); r += 2 * kLanes) {
                    typename M::Vec qj[2];
                    float4 sh[2];
                    uint32_t j[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        j[u] = entry_particle(e[u]);
                        qj[u] = load_vec<M>(q4, j[u]);
                        sh[u] = shift[e[u] >> kEntryBits];
                    }
                    e[0] = entry(r + 2 * kLanes);
                    e[1] = entry(r + 3 * kLanes);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const float d[3] = {(qi.x - qj[u].x) + sh[u].x, (qi.y - qj[u].y) + sh[u].y,
                                            (qi.z - qj[u].z) + sh[u].z};
                        const float r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
                        float out[NV];
                        term(j[u], j[u] == (uint32_t)i, qi, qj[u], d, r2, out);
                        for (int v = 0; v < NV; ++v) acc[v] = acc[v] + moved<0x00>(out[v]);
                        for (int v = 0; v < NV; ++v) acc[v] = acc[v] + moved<0x55>(out[v]);
                        for (int v = 0; v < NV; ++v) acc[v] = acc[v] + moved<0xaa>(out[v]);
                        for (int v = 0; v < NV; ++v) acc[v] = acc[v] + moved<0xff>(out[v]);
                    }
                }
            } while (next_part());
            for (int v = 0; v < NV; ++v)
                if (s == (uint32_t)v) mine = acc[v];
        }
        for (uint64_t todo = __ballot(over && s == 0u); todo; todo &= todo - 1ull) {
            const int l = __builtin_ctzll(todo);
            const int64_t at = (int64_t)lane_of((uint32_t)i, l);
            Real sum[NV];
            Term whole = term;
            direct(at, whole, sum);
            if (lane / kLanes == l / kLanes)
                for (int v = 0; v < NV; ++v)
                    if (s == (uint32_t)v) mine = sum[v];
        }
        return mine;
    }
};

// particle of this lane's group (past the last one: the last, live = false)
template <class M>
__device__ __forceinline__ int64_t partner_particle(const DevParams &P, uint32_t blk, bool &live)
{
    const int64_t i = (int64_t)blk * (blockDim.x / M::kLanes) + threadIdx.x / M::kLanes;
    live = i < P.n;
    return live ? i : P.n - 1;
}

// ---------------------------------------------------------------- forces
struct ForcesArgs {
    PartnerArgs a;           // records (x, y, z, Pi)
    double *f, *p;
    int half_kick;
};

// m^2 (Pi_i + Pi_j) F_ij r_ij
template <class M, bool LUCY>
struct ForceTerm {
    typedef typename M::Real Real;
    const DevParams &P;
    const Real ms;
    __device__ __forceinline__ void at(int64_t) {}
    __device__ __forceinline__ void operator()(uint32_t, bool own, const typename M::Vec &qi,
                                               const typename M::Vec &qj, const Real d[3],
                                               Real r2, Real out[3]) const
    {
        Real sc = ms * (qi.w + qj.w) * M::template force<LUCY>(P, r2);
        asm volatile("" : "+v"(sc));   // (a select, no branch around the factors)
        sc = own ? (Real)0 : sc;
        for (int x = 0; x < 3; ++x) out[x] = sc * d[x];
    }
};

template <class M, bool LUCY>
__device__ __forceinline__ void forces_body(const ForcesArgs &g, uint32_t blk)
{
    __shared__ float4 shift[4][M::kShiftEverywhere ? NNB : 1];
    const DevParams &P = g.a.P;
    bool live;
    const int64_t i = partner_particle<M>(P, blk, live);
    const int lane = threadIdx.x & 63;
    PartnerSums<M, 3, ForceTerm<M, LUCY>> sums{g.a, P, shift[threadIdx.x >> 6], lane,
                                               (uint32_t)lane % M::kLanes};
    const double f = (double)sums.run(i, live, ForceTerm<M, LUCY>{P, M::force_scale(P)});
    if (!live || sums.s >= 3u) return;
    const int64_t at = sums.s * P.n + i;
    g.f[at] = f;
    if (g.half_kick) g.p[at] += 0.5 * P.dt * f;
}

// ---------------------------------------------------------------- launches
// Density: in launches recorded for a batch all boxes share the GPU, and take the
// form of large ones (the two agree bit for bit); a box on its own: four waves per cell up
// to 2^10 cells, one per SIMD of the GPU (384 cells: 25 us against 50; 1728 cells: 53
// against 54; 7128: 102 against 73).
constexpr int64_t kSplitMaxCells = 1 << 10;
// A lane per particle from 2^15 cells of fewer than four particles on average on: 64000
// cells of 0.25, 1, 2, 3, 3.9 particles 38, 53, 73, 98, 125 us, a wave per cell 64, 78, 91,
// 109, 124; 13824 cells, whose waves all fit at once, 32, 45, 58, 69 against 21, 24, 27, 32.
constexpr int64_t kSparsePerCell = 4, kSparseMinCells = 1 << 15;

template <class M, bool LUCY>
__device__ __forceinline__ void density_body(const DensityArgs &a, uint32_t blk)
{
    __shared__ DensityLds<M, false> lds;
    density_cells<M, LUCY, false>(a, blk, lds);
}
template <class M, bool LUCY, bool SPLIT>
__global__ __launch_bounds__(64 * kCellWaves, SPLIT ? 1 : M::kDensityOcc) void k_density(DensityArgs a)
{
    __shared__ DensityLds<M, SPLIT> lds;
    density_cells<M, LUCY, SPLIT>(a, xcd_block(blockIdx.x, gridDim.x), lds);
}
template <class M, bool LUCY>
__global__ __launch_bounds__(256) void k_density_sparse(DensityArgs a)
{
    density_sparse<M, LUCY>(a, xcd_block(blockIdx.x, gridDim.x));
}
template <class M, bool LUCY>
__global__ __launch_bounds__(64, M::kDensityOcc) void k_density_dense(DensityArgs)
{
    density_dense<M, LUCY>(kernel_argument<DensityArgs>(), xcd_block(blockIdx.x, gridDim.x));
}
template <class M, bool LUCY>
__global__ __launch_bounds__(256) void k_forces(ForcesArgs g)
{
    forces_body<M, LUCY>(g, xcd_block(blockIdx.x, gridDim.x));
}

// the multi-box forms of a model and kernel
struct DensityMulti {
    MultiKernel cells, sparse, dense;
};
template <class M, bool LUCY>
int launch_density(sdpd_ctx *c, const DensityArgs &args, const DensityMulti &multi)
{
    if (c->ncell >= kSparseMinCells && c->n < kSparsePerCell * c->ncell) {
        const int rc = launch_or_record(c, k_density_dense<M, LUCY>, multi.dense,
                                        (unsigned)((c->n + kHeads - 1) / kHeads), 64, 0, args);
        if (rc) return rc;
        return launch_or_record(c, k_density_sparse<M, LUCY>, multi.sparse,
                                (unsigned)((c->n + 255) / 256), 256, 0, args);
    }
    if (c->ncell <= kSplitMaxCells && !c->rec) {
        hipLaunchKernelGGL((k_density<M, LUCY, true>), dim3((unsigned)c->ncell),
                           dim3(64 * kCellWaves), 0, c->stream, args);
        return check_hip(hipGetLastError());
    }
    return launch_or_record(c, k_density<M, LUCY, false>, multi.cells,
                            (unsigned)((c->ncell + kCellWaves - 1) / kCellWaves),
                            64 * kCellWaves, 0, args);
}
template <class M, bool LUCY>
int launch_forces(sdpd_ctx *c, const ForcesArgs &args, MultiKernel multi)
{
    return launch_or_record(c, k_forces<M, LUCY>, multi,
                            (unsigned)((c->n + 256 / M::kLanes - 1) / (256 / M::kLanes)), 256, 0, args);
}

inline PartnerArgs partner_args(const sdpd_ctx *c, const void *q4)
{
    return PartnerArgs{c->dp, q4, c->cell_sorted, c->cell_start, c->list, c->list_count,
                       c->list_len, c->list_cap};
}

}  // namespace sdpd
