// Pairwise fluctuation/dissipation sweep with the Metropolis correction of
// Faure & Stoltz: the proposal of eq. (proposal) (the Ornstein-Uhlenbeck
// step of eq. ssa-ou written in the relative velocity), the energy update of
// eq. (proposal-update), the energy bound of eq. (energy-bound) and the
// log-ratio of eq. (metropolis-ratio) (Sec. 3.3.2); AMS and SSA as modes.
//
// Order of the pair updates.  Every active pair (r < h) has the key
// (phase, round): phase 0 = pairs inside one cell, phase 1 + 8 o + pi =
// pairs between a cell A of coordinate parity pi and A + delta_o (o-th of
// the 13 forward offsets); round = slot_A XOR slot_B.  The sweep is the
// sequential application in ascending key.  Inside one phase the tasks
// (one cell, or one cell pair) share no particle, and inside a task two
// pairs of one round share no particle, so any schedule that keeps the key
// order between pairs sharing a particle gives the same result.
//
// GPU schedule.  The scheduling pass (schedule.hip) has stored, for every
// task, its active pairs with their conflict level.  A workgroup (one wave)
// takes a range of consecutive tasks of one phase, sorts the range's pairs by
// level, forms a record of each pair (unit vector, friction exponent, random
// draws: everything that does not change during the sweep) at full lane
// occupancy in that order, stages in LDS the momenta and energies of the
// particles that take part, and applies the pairs of one level (which share no
// particle) 64 at a time, the records of the next step in flight meanwhile.
// The number of level steps of a batch is set by its deepest task (the longest
// chain of pairs that share a particle, in round order), not by its size, so a
// step holds 28 pairs on average: what can be worked out beforehand leaves the
// steps.
//
// What bounds it (2^20 particles, 38 million pairs, MI355X): VALU issue.  A
// step at three waves per SIMD takes as much longer as there are waves (3,100
// against 4,500 cycles at two), so only fewer instructions help: the records
// with the pair update in scalars of the pair (fd_pair) took the step from
// ~560 to ~320 VALU instructions and the sweep from 2.285 to 1.96 ms, constants
// kept out of the way of the steps (fd_math.hpp, `reread`) and FP64 FMAs
// without coefficient copies to 1.90 ms, three waves per SIMD in 168 registers
// to 1.81 ms.  Forming the records in a launch of its own, for all ranges
// before the sweep, was slower for large boxes (1.07 + 1.46 ms: 2.4 GB of
// records go through HBM instead of the workgroups' slices in the last-level
// cache), faster only for small ones (see fd_levels).
//
// Phases that touch disjoint cells commute.  Phase 1 + 8 o + pi touches the
// cells of parity pi (as A) and pi ^ b_o (as B = A + delta_o, b_o the parity
// bits that delta_o flips; the number of cells per axis is even, so this
// holds across the periodic boundary).  Each phase is given the level
// 1 + the largest level of the earlier phases whose parity sets intersect
// its own; the phases of one level form a group.  For the 13 forward offsets
// this gives 26 groups of 4 phases, each touching every cell exactly once;
// with phase 0, 27 groups.  The whole sweep is one persistent launch: the
// task ranges of all groups, in group order, are handed out by an atomic
// counter, and a range of group g waits only until every cell it touches
// has been released by group g - 1 (per-cell epochs), so the groups overlap
// instead of draining one launch before the next.  Every pair of phases
// whose order is exchanged touches disjoint particles, so the result equals
// the sweep in key order bit for bit.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <memory>
#include <vector>

#include "fd_math.hpp"
#include "tasks.hpp"

namespace sdpd {

constexpr int FD_NLVL = 64;        // levels of a task are 1..64
constexpr int FD_EPL = 16;         // pair entries per lane held in registers
constexpr int FD_PPL = 8;          // particle-list entries per lane per staging pass
constexpr int FD_MAXPH = 4;        // phases per launch

struct FdLaunch {
    int nph;
    int cap_p, cap_e;                // LDS capacity: particles, pair entries
    int64_t task_base[FD_MAXPH];     // index of the phase's first task in sweep order
    int64_t ntasks[FD_MAXPH];
    int64_t tpw[FD_MAXPH];           // tasks per workgroup
    int64_t wg_end[FD_MAXPH];        // cumulative workgroup counts
};

// dynamic LDS layout: gidx[cap_p] and the level tables (32-bit), then one area
// that holds first the sorted pair list [cap_e] (32-bit) and, once the pairs'
// records are formed, the state (p_x, p_y, p_z, eps)[cap_p] (doubles)
constexpr int FD_TABLE_WORDS = 2 * (FD_NLVL + 2);
__host__ __device__ inline int fd_lds_area(int cap_p)   // byte offset of the shared area
{
    return (4 * (cap_p + FD_TABLE_WORDS) + 15) & ~15;
}
__host__ __device__ inline size_t fd_lds_bytes(int cap_p, int cap_e)
{
    const size_t st = (size_t)32 * cap_p, so = (size_t)4 * cap_e;
    return (size_t)fd_lds_area(cap_p) + (st > so ? st : so);
}
// what a tuning is checked against (sdpd_tune): the list beside the state
inline size_t fd_lds_checked_bytes(int cap_p, int cap_e)
{
    return (size_t)36 * cap_p + (size_t)4 * cap_e + 1320;
}

struct FdLds {
    uint32_t *gidx, *hist, *cur;
    uint32_t *sorted;   // A-side | B-side << 16
    double2 *st;        // (p_x, p_y), (p_z, eps) per particle; the same memory
    __device__ __forceinline__ FdLds(unsigned char *lds, int cap_p)
    {
        gidx = (uint32_t *)lds;
        hist = gidx + cap_p;
        cur = hist + (FD_NLVL + 2);
        sorted = (uint32_t *)(lds + fd_lds_area(cap_p));
        st = (double2 *)sorted;
    }
};

constexpr uint64_t POS_MASK = (1ull << 25) - 1ull;   // list position field of a pair entry

// The records of one batch (PairRec): four planes of n entries of 16 bytes
struct RecPlanes {
    double2 *p;
    int64_t n;
    __device__ __forceinline__ void store(int e, const PairRec &r) const
    {
        p[e] = make_double2(r.ex, r.ey);
        p[n + e] = make_double2(r.ez, r.y);
        p[2 * n + e] = make_double2(r.G0, r.G1);
        p[3 * n + e] = make_double2(r.G2, __hiloint2double((int)r.ij, (int)r.u));
    }
    __device__ __forceinline__ PairRec load(int e) const
    {
        const double2 a = p[e], b = p[n + e], c = p[2 * n + e], d = p[3 * n + e];
        return PairRec{a.x, a.y, b.x, b.y, c.x, c.y, d.x, (uint32_t)__double2loint(d.y),
                       (uint32_t)__double2hiint(d.y)};
    }
};

// Momenta and energies are the state that workgroups hand on to each other.
// COHERENT (the one-launch sweep): another workgroup of the same kernel, on
// any XCD, may have written them, so they are read and written with
// agent-scope atomic loads and stores (coherent across the XCDs' L2 caches,
// with no cache flush); otherwise (one launch per group) plain accesses.
template <bool COHERENT>
__device__ __forceinline__ double state_load(const double *ptr)
{
    if (COHERENT) return __hip_atomic_load(ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *ptr;
}

template <bool COHERENT>
__device__ __forceinline__ void state_store(double *ptr, double v)
{
    if (COHERENT) __hip_atomic_store(ptr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *ptr = v;
}

// Arguments every range of the sweep reads or writes.
struct FdArgs {
    const double4 *qrho;
    double *p, *eps;
    const uint32_t *id, *pair_off, *part_off;
    const uint64_t *pairs;
    const uint32_t *part_list;
    uint32_t pair_cap, part_cap;
    const uint64_t *dstep;
    double dt, y_c;         // time step of the sweep; prefactor of a pair's exponent
    double2 *rec;           // pair records, batch by batch
    int64_t rec_stride;     // one-launch sweep: 16-byte units of a workgroup's slice
    uint16_t *lvl;          // records formed by k_fd_records: per batch (at its first task): end of each level, FD_NLVL entries
    uint32_t *err;
};

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, int lane)   // uniform lane
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Range b of the launch L (consecutive tasks of one of its phases): lane t
// holds the offsets of task t (pair entries and particle-list entries, first
// and end; lanes past the range: empty tasks).
struct FdRange {
    int R;                       // tasks, at most one per lane
    int64_t T0;                  // the first one, in sweep order
    uint32_t e_lo, e_hi, p_lo, p_hi;
    uint32_t phase_p0;           // first particle-list entry of the phase
    uint32_t rec0;               // record of pair entry e: rec0 + e
    bool ok;                     // the schedule holds all of its entries
};

__device__ __forceinline__ FdRange fd_range_of(const FdLaunch &L, int64_t b, const FdArgs &A,
                                               bool group_records)
{
    static_assert(FD_WAVES == 1, "lane = thread: offsets and levels are held per lane");
    const int tid = threadIdx.x;
    FdRange r;
    int k_ph = 0;
    while (k_ph + 1 < L.nph && b >= L.wg_end[k_ph]) ++k_ph;
    if (k_ph > 0) b -= L.wg_end[k_ph - 1];
    const int64_t tpw = L.tpw[k_ph], ntasks = L.ntasks[k_ph], task_base = L.task_base[k_ph];
    const int64_t t0 = b * tpw;
    r.R = (int)(t0 + tpw < ntasks ? tpw : ntasks - t0);
    r.T0 = task_base + t0;
    const int64_t lo = r.T0 + min(tid, r.R), hi = r.T0 + min(tid + 1, r.R);
    r.e_lo = A.pair_off[lo];
    r.p_lo = A.part_off[lo];
    r.e_hi = A.pair_off[hi];
    r.p_hi = A.part_off[hi];
    r.phase_p0 = A.part_off[task_base];
    r.rec0 = 0;
    if (group_records) {   // place among the entries of the group's phases
        for (int k = 0; k < k_ph; ++k)
            r.rec0 += A.pair_off[L.task_base[k] + L.ntasks[k]] - A.pair_off[L.task_base[k]];
        r.rec0 -= A.pair_off[task_base];
    }
    r.ok = lane_u32(r.e_hi, 63) <= A.pair_cap && lane_u32(r.p_hi, 63) <= A.part_cap;
    return r;
}

// A batch of consecutive tasks k0 .. k - 1 of a range that fits the LDS
// capacities (scalar work on the lanes' offsets; finding its end with a ballot
// was slower, 2.08 against 1.95 ms a sweep at 2^20 particles, through the
// registers it held); a task with more pairs than the list forms one of its
// own (oversized).
struct FdBatch {
    int k0, k, npr, np;          // tasks, pairs, particles
    uint32_t e_begin, p_begin;
    bool oversized;
};

__device__ __forceinline__ FdBatch fd_next_batch(const FdRange &r, int k, int CP, int CE)
{
    FdBatch t;
    t.k0 = k;
    t.oversized = false;
    t.e_begin = lane_u32(r.e_lo, k);
    t.p_begin = lane_u32(r.p_lo, k);
    while (k < r.R) {
        const int c = (int)(lane_u32(r.e_hi, k) - lane_u32(r.e_lo, k));
        const int np_new = (int)(lane_u32(r.p_hi, k) - t.p_begin);
        const int npr_new = (int)(lane_u32(r.e_hi, k) - t.e_begin);
        if (k > t.k0 && c > 0 && (np_new > CP || npr_new > CE)) break;
        t.oversized = c > CE;   // only possible as the first task of a batch
        ++k;
        if (t.oversized) break;
    }
    t.k = k;
    t.npr = (int)(lane_u32(r.e_hi, k - 1) - t.e_begin);
    t.np = (int)(lane_u32(r.p_hi, k - 1) - t.p_begin);
    return t;
}

// global indices of the particles that take part in a pair of the batch
__device__ __forceinline__ void fd_load_indices(const FdArgs &A, const FdBatch &t, const FdLds &S)
{
    const uint32_t *__restrict__ part_list = A.part_list;
    const int tid = threadIdx.x;
    for (int base = 0; base < t.np; base += FD_PPL * FD_THREADS) {
        uint32_t gl[FD_PPL];
#pragma unroll
        for (int q = 0; q < FD_PPL; ++q) {
            const int l = base + q * FD_THREADS + tid;
            gl[q] = l < t.np ? part_list[t.p_begin + l] : 0u;
        }
#pragma unroll
        for (int q = 0; q < FD_PPL; ++q) {
            const int l = base + q * FD_THREADS + tid;
            if (l < t.np) S.gidx[l] = gl[q];
        }
    }
    __syncthreads();
}

// Counting sort of the batch's entries of the levels lo .. hi into S.sorted.
// hi = FD_NLVL, or for an oversized batch the last level up to which the list
// holds them.  Returns the inclusive prefix over the levels (lane x: level
// x + 1).
__device__ __forceinline__ uint32_t fd_sort_window(const FdArgs &A, const FdBatch &t,
                                                   uint32_t rel0, const FdLds &S, int CE, int lo,
                                                   int &hi)
{
    const uint64_t *__restrict__ pairs = A.pairs;
    const int tid = threadIdx.x, npr = t.npr, np = t.np;
    const uint32_t e_begin = t.e_begin;
    hi = FD_NLVL;
    S.hist[tid + 1] = 0u;
    __syncthreads();
    if (t.oversized) {
        for (int e = tid; e < npr; e += FD_THREADS) {
            const int lv = (int)(pairs[e_begin + e] >> 50);
            if (lv >= 1 && lv <= FD_NLVL) atomicAdd(&S.hist[lv], 1u);
        }
        __syncthreads();
        int acc = 0;
        for (hi = lo; hi <= FD_NLVL; ++hi) {
            if (acc + (int)S.hist[hi] > CE) break;
            acc += (int)S.hist[hi];
        }
        --hi;
        hi = hi < lo ? lo : hi;   // one level (<= 64 pairs) always fits
        __syncthreads();
        S.hist[tid + 1] = 0u;
        __syncthreads();
    }
    // histogram pass, prefix, scatter pass.  Entries stay in registers
    // (FD_EPL per lane) between the passes unless the batch needs several.
    constexpr int EP = FD_EPL * FD_THREADS;
    uint64_t ebuf[FD_EPL];
    const bool one_pass = npr <= EP;
    for (int base = 0; base < npr; base += EP) {
#pragma unroll
        for (int q = 0; q < FD_EPL; ++q) {
            const int x = base + q * FD_THREADS + tid;
            ebuf[q] = x < npr ? pairs[e_begin + x] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < FD_EPL; ++q) {
            const uint64_t e = ebuf[q];
            const int lv = (int)(e >> 50);
            const int li = (int)((uint32_t)(e & POS_MASK) - rel0);
            const int lj = (int)((uint32_t)((e >> 25) & POS_MASK) - rel0);
            if (lv >= lo && lv <= hi && lv <= FD_NLVL && li >= 0 && li < np && lj >= 0 && lj < np)
                atomicAdd(&S.hist[lv], 1u);
        }
    }
    __syncthreads();
    const uint32_t h = S.hist[tid + 1];
    uint32_t incl = h;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)incl, off);
        if (tid >= off) incl += v;
    }
    S.cur[tid + 1] = incl - h;
    __syncthreads();
    for (int base = 0; base < npr; base += EP) {
        if (!one_pass) {
#pragma unroll
            for (int q = 0; q < FD_EPL; ++q) {
                const int x = base + q * FD_THREADS + tid;
                ebuf[q] = x < npr ? pairs[e_begin + x] : 0ull;
            }
        }
#pragma unroll
        for (int q = 0; q < FD_EPL; ++q) {
            const uint64_t e = ebuf[q];
            const int lv = (int)(e >> 50);
            const int li = (int)((uint32_t)(e & POS_MASK) - rel0);
            const int lj = (int)((uint32_t)((e >> 25) & POS_MASK) - rel0);
            if (lv >= lo && lv <= hi && lv <= FD_NLVL && li >= 0 && li < np && lj >= 0 &&
                lj < np) {
                const uint32_t pos = atomicAdd(&S.cur[lv], 1u);
                if (pos < (uint32_t)CE) S.sorted[pos] = (uint32_t)li | ((uint32_t)lj << 16);
            }
        }
    }
    __syncthreads();
    return incl;
}

// Records of the ntot sorted entries into planes first, first + 1, ..., all
// lanes busy.  The ids also orient each pair (i = smaller id); the gathers of
// the next 64 entries are in flight while these are worked out.
template <int K>
__device__ __forceinline__ void fd_form_records(const DevParams &P, const FdArgs &A,
                                                const FdLds &S, int ntot, const RecPlanes &rec,
                                                int first)
{
    const double4 *__restrict__ qrho = A.qrho;
    const uint32_t *__restrict__ id = A.id;
    const uint32_t step = (uint32_t)*A.dstep;   // step index of the Philox counter
    ColdTable *tab = cold(kDrawTab);
    const int tid = threadIdx.x;
    uint32_t pr, ida, idb;
    double4 qa, qb;
    auto gather = [&](int e) {
        pr = S.sorted[min(e, ntot - 1)];
        const uint32_t ga = S.gidx[pr & 0xFFFFu], gb = S.gidx[pr >> 16];
        ida = id[ga];
        idb = id[gb];
        qa = qrho[ga];
        qb = qrho[gb];
    };
    if (ntot > 0) gather(tid);
    for (int base = 0; base < ntot; base += FD_THREADS) {
        const int e = base + tid;
        const bool swap = ida > idb;
        const uint32_t ij = swap ? (pr >> 16) | (pr << 16) : pr;
        const uint32_t id0 = swap ? idb : ida, id1 = swap ? ida : idb;
        const double4 a = qa, b = qb;
        if (base + FD_THREADS < ntot) gather(e + FD_THREADS);
        PairRec g = pair_record<K>(P, A.y_c, step, id0, id1, a, b, tab);
        // e_ij of the swapped pair (exact)
        g.ex = swap ? -g.ex : g.ex;
        g.ey = swap ? -g.ey : g.ey;
        g.ez = swap ? -g.ez : g.ez;
        g.ij = ij;
        if (e < ntot) rec.store(first + e, g);
    }
    __syncthreads();
}

// Momenta and energies of the batch staged over the list; the loads of several
// particles issue before their LDS writes (an LDS write between two atomic
// loads makes the second wait).
template <bool COHERENT>
__device__ __forceinline__ void fd_stage(const FdArgs &A, int64_t n, int np, const FdLds &S)
{
    const double *p = A.p, *eps = A.eps;
    const int tid = threadIdx.x;
    constexpr int SPL = 4;
    for (int base = 0; base < np; base += SPL * FD_THREADS) {
        double v[SPL][4];
        int64_t gi[SPL];
#pragma unroll
        for (int q = 0; q < SPL; ++q) gi[q] = S.gidx[min(base + q * FD_THREADS + tid, np - 1)];
#pragma unroll
        for (int q = 0; q < SPL; ++q) {
            v[q][0] = state_load<COHERENT>(p + gi[q]);
            v[q][1] = state_load<COHERENT>(p + n + gi[q]);
            v[q][2] = state_load<COHERENT>(p + 2 * n + gi[q]);
            v[q][3] = state_load<COHERENT>(eps + gi[q]);
        }
#pragma unroll
        for (int q = 0; q < SPL; ++q) {
            const int l = base + q * FD_THREADS + tid;
            if (l < np) {
                S.st[2 * l] = make_double2(v[q][0], v[q][1]);
                S.st[2 * l + 1] = make_double2(v[q][2], v[q][3]);
            }
        }
    }
    __syncthreads();
}

template <bool COHERENT>
__device__ __forceinline__ void fd_write_back(const FdArgs &A, int64_t n, int np, const FdLds &S)
{
    double *p = A.p, *eps = A.eps;
    for (int l = threadIdx.x; l < np; l += FD_THREADS) {
        const int64_t g = S.gidx[l];
        const double2 a = S.st[2 * l], c = S.st[2 * l + 1];
        state_store<COHERENT>(p + g, a.x);
        state_store<COHERENT>(p + n + g, a.y);
        state_store<COHERENT>(p + 2 * n + g, c.x);
        state_store<COHERENT>(eps + g, c.y);
    }
    __syncthreads();
}

// The pair updates: steps of at most 64 records of one level in ascending
// order (ends: lane x holds the end of level x + 1); the records of step k + 1
// are in flight while step k runs.
template <int K>
__device__ __forceinline__ void fd_run_levels(const DevParams &P, double dt, int ends,
                                              const RecPlanes &rec, const FdLds &S, FdCount &cnt,
                                              bool &negeps)
{
    const int tid = threadIdx.x;
    const int ntot = __builtin_amdgcn_readlane(ends, FD_NLVL - 1);
    const int last = max(ntot - 1, 0);
    int lev = 0, pos = -FD_THREADS, end = 0;
    auto advance = [&] {
        pos += FD_THREADS;
        while (pos >= end && end < ntot) {   // the next level that is not empty
            pos = end;
            end = __builtin_amdgcn_readlane(ends, lev);
            ++lev;
        }
    };
    const PairRegs<K == 2> c(P);
    advance();
    PairRec g0 = rec.load(min(pos + tid, last));
    bool v0 = pos + tid < end;
    while (pos < end) {
        advance();
        const PairRec g1 = rec.load(min(pos + tid, last));
        const bool v1 = pos + tid < end;
        if (v0) fd_pair<K>(P, c, dt, g0, S.st, cnt, negeps);
        __syncthreads();
        g0 = g1;
        v0 = v1;
    }
}

// One range of the sweep: batch by batch its entries sorted, its records
// formed, its state staged, the levels applied, the state written back.
// K: 0 = general, 1 = the common case (EMS, Lucy kernel, zeta = 0) fixed at
// compile time, 2 = that case with the FP32 proposal of mixed precision.
// Only this workgroup reads the records: they go to its own slice (one-launch
// sweep) or to the batch's place among the entries of its group, which touches
// every cell once and so holds at most 32 pairs per particle (two cells of a
// and b particles, at most 64 each, have a b <= 32 (a + b) pairs).
// wait() is called once, before the first access to momenta and energies:
// everything before it (entries, lists, ids, positions, the records) is fixed
// during the sweep, so the level sort and the records of a range overlap the
// wait for its predecessors.
template <int K, bool COHERENT, class Wait>
__device__ __forceinline__ void fd_range(const DevParams &P, const FdLaunch &L, int64_t b,
                                         unsigned char *lds, const FdArgs &A, FdCount &cnt,
                                         bool &negeps, Wait &wait)
{
    const int CP = L.cap_p, CE = L.cap_e;
    const FdLds S(lds, CP);
    const FdRange r = fd_range_of(L, b, A, !COHERENT);
    if (!r.ok) {   // schedule incomplete
        if (threadIdx.x == 0) atomicOr(A.err, ERR_PAIRCAP);
        return;
    }
    for (int k = 0; k < r.R;) {
        const FdBatch t = fd_next_batch(r, k, CP, CE);
        k = t.k;
        if (t.npr == 0) continue;
        const FdArgs &B = reread(A);
        const RecPlanes rec =
            COHERENT ? RecPlanes{B.rec + (int64_t)blockIdx.x * B.rec_stride, min(t.npr, CE)}
                     : RecPlanes{B.rec + 4 * (int64_t)(uint32_t)(r.rec0 + t.e_begin), t.npr};
        fd_load_indices(B, t, S);
        // windows of levels: one, unless a single task overflows the list
        for (int lo = 1, hi; lo <= FD_NLVL; lo = hi + 1) {
            const uint32_t ends = fd_sort_window(B, t, t.p_begin - r.phase_p0, S, CE, lo, hi);
            fd_form_records<K>(reread(P), B, S, min((int)lane_u32(ends, FD_NLVL - 1), CE), rec, 0);
            wait();
            fd_stage<COHERENT>(reread(A), reread(P).n, t.np, S);
            fd_run_levels<K>(reread(P), reread(A).dt, min((int)ends, CE), rec, S, cnt, negeps);
            fd_write_back<COHERENT>(reread(A), reread(P).n, t.np, S);
            if (!t.oversized) break;
            // the next window stages what this one has written
            __builtin_amdgcn_s_waitcnt(0);
        }
    }
}

// Small boxes with one launch per group: the records and level ends of every
// range by a launch of their own (fd_records), so that the 27 dependent
// launches only stage, apply the levels and write back (fd_levels).
template <int K>
__device__ __forceinline__ void fd_records(const DevParams &P, const FdLaunch &L, int64_t b,
                                           unsigned char *lds, const FdArgs &A)
{
    const int CP = L.cap_p, CE = L.cap_e, tid = threadIdx.x;
    const FdLds S(lds, CP);
    const FdRange r = fd_range_of(L, b, A, false);
    if (!r.ok) {   // schedule incomplete
        if (tid == 0) atomicOr(A.err, ERR_PAIRCAP);
        return;
    }
    for (int k = 0; k < r.R;) {
        const FdBatch t = fd_next_batch(r, k, CP, CE);
        k = t.k;
        if (t.npr == 0) continue;
        const RecPlanes rec{A.rec + 4 * (int64_t)t.e_begin, t.npr};
        fd_load_indices(A, t, S);
        int done = 0;        // records of the levels before lo
        uint32_t ends = 0;
        for (int lo = 1, hi; lo <= FD_NLVL; lo = hi + 1) {
            const uint32_t incl = fd_sort_window(A, t, t.p_begin - r.phase_p0, S, CE, lo, hi);
            const int ntot = min((int)lane_u32(incl, FD_NLVL - 1), CE);
            if (tid + 1 >= lo) ends = (uint32_t)done + min(incl, (uint32_t)CE);
            fd_form_records<K>(P, A, S, ntot, rec, done);
            done += ntot;
            if (!t.oversized) break;
        }
        A.lvl[(r.T0 + t.k0) * FD_NLVL + tid] = (uint16_t)ends;
    }
}

template <int K>
__device__ __forceinline__ void fd_levels(const DevParams &P, const FdLaunch &L, int64_t b,
                                          unsigned char *lds, const FdArgs &A, FdCount &cnt,
                                          bool &negeps)
{
    const int CP = L.cap_p, CE = L.cap_e;
    const FdLds S(lds, CP);
    const FdRange r = fd_range_of(L, b, A, false);
    if (!r.ok) return;   // reported by the record pass
    for (int k = 0; k < r.R;) {
        const FdBatch t = fd_next_batch(r, k, CP, CE);
        k = t.k;
        if (t.npr == 0) continue;
        const RecPlanes rec{A.rec + 4 * (int64_t)t.e_begin, t.npr};
        const int ends = (int)A.lvl[(r.T0 + t.k0) * FD_NLVL + threadIdx.x];
        fd_load_indices(A, t, S);
        fd_stage<false>(A, P.n, t.np, S);
        fd_run_levels<K>(P, A.dt, ends, rec, S, cnt, negeps);
        fd_write_back<false>(A, P.n, t.np, S);
    }
}

// counters of a workgroup: one atomic per counter
__device__ __forceinline__ void fd_flush_counters(const FdCount &cnt, bool negeps,
                                                  unsigned long long *counters, uint32_t *err)
{
    const int lane = threadIdx.x & 63;   // one flush per wave
    const uint32_t v0 = wave_sum_u32(cnt.proposed), v1 = wave_sum_u32(cnt.rej_energy);
    const uint32_t v2 = wave_sum_u32(cnt.rej_ratio), v3 = wave_sum_u32(cnt.marginal);
    const uint32_t v4 = wave_sum_u32(cnt.negeps);
    const bool any_neg = __ballot(negeps) != 0ull;
    if (lane == 0) {
        if (v0) atomicAdd(&counters[CNT_PROPOSED], (unsigned long long)v0);
        if (v1) atomicAdd(&counters[CNT_REJ_ENERGY], (unsigned long long)v1);
        if (v2) atomicAdd(&counters[CNT_REJ_RATIO], (unsigned long long)v2);
        if (v3) atomicAdd(&counters[CNT_MARGINAL], (unsigned long long)v3);
        if (v4) atomicAdd(&counters[CNT_NEGEPS], (unsigned long long)v4);
        if (any_neg) atomicOr(err, ERR_NEGEPS);
    }
}

// one launch per group: workgroup b applies range b of L
struct FdPhaseArgs {
    const DevParams *Pp;
    FdLaunch L;
    FdArgs A;
    unsigned long long *counters;
};
template <int K>
__device__ __forceinline__ void fd_phase_body(const FdPhaseArgs &a, uint32_t blk)
{
    extern __shared__ __align__(16) unsigned char lds[];
    FdCount cnt = {0u, 0u, 0u, 0u, 0u};
    bool negeps = false;
    auto no_wait = [] {};
    fd_range<K, false>(*a.Pp, a.L, (int64_t)blk, lds, a.A, cnt, negeps, no_wait);
    fd_flush_counters(cnt, negeps, a.counters, a.A.err);
}
template <int K>
__global__ __launch_bounds__(FD_THREADS) void k_fd_phase(FdPhaseArgs)
{
    fd_phase_body<K>(kernel_argument<FdPhaseArgs>(), blockIdx.x);
}
SDPD_MULTI_KERNEL(k_fd_phase_gen_multi, FdPhaseArgs, fd_phase_body<0>, FD_THREADS)
SDPD_MULTI_KERNEL(k_fd_phase_fast_multi, FdPhaseArgs, fd_phase_body<1>, FD_THREADS)
SDPD_MULTI_KERNEL(k_fd_phase_mix_multi, FdPhaseArgs, fd_phase_body<2>, FD_THREADS)

// the same with the records already formed (k_fd_records)
template <int K>
__global__ __launch_bounds__(FD_THREADS) void k_fd_levels(FdPhaseArgs a)
{
    extern __shared__ __align__(16) unsigned char lds[];
    FdCount cnt = {0u, 0u, 0u, 0u, 0u};
    bool negeps = false;
    fd_levels<K>(*a.Pp, a.L, (int64_t)blockIdx.x, lds, a.A, cnt, negeps);
    fd_flush_counters(cnt, negeps, a.counters, a.A.err);
}

// The whole sweep in one launch.  Its ranges, group by group (group 0 =
// phase 0, then the groups of mutually disjoint phases; inside a group in
// the order of `order`), are handed out by an atomic counter, so a range is
// only taken by a running workgroup and every range it waits for was taken
// before it.  Every group touches every
// cell exactly once, so epoch[c] = the number of groups done on cell c: a
// range of group g waits until its cells have epoch g, and sets them to
// g + 1 once its momenta and energies are written (stores completed first).
// A wait normally lasts microseconds, but when many queues share the GPU a
// workgroup holding a needed range can be descheduled for a long time (tens
// of milliseconds were measured with 32 queues), so the wait is bounded in
// time, not in polls: after kWaitTicks of the constant 100 MHz clock it
// reports ERR_STALL and goes on, so every workgroup ends.
constexpr int FD_MAXGROUPS = 32;
struct FdSweep {
    int ngroups;
    uint32_t nitems;
    uint32_t group_end[FD_MAXGROUPS];   // cumulative ranges per group
    FdLaunch launch[FD_MAXGROUPS];
};
constexpr uint64_t kWaitTicks = 20ull * 100000000ull;   // 20 s

// The records of all ranges of the sweep, one workgroup per range.
template <int K>
__global__ __launch_bounds__(FD_THREADS) void k_fd_records(const DevParams *__restrict__ Pp,
                                                           const FdSweep *__restrict__ SW,
                                                           FdArgs A)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const uint32_t it = blockIdx.x;
    int g = 0;
    while (it >= SW->group_end[g]) ++g;
    fd_records<K>(*Pp, SW->launch[g], (int64_t)(it - (g > 0 ? SW->group_end[g - 1] : 0u)), lds, A);
}

// One range of the one-launch sweep: range b of group g, waiting until the
// cells of its tasks have epoch g and setting them to g + 1 afterwards.
template <int K>
__device__ __forceinline__ void fd_flow_range(const DevParams &P, const FdLaunch &L, int g,
                                              int64_t b, const FdArgs &A, uint32_t *epoch,
                                              unsigned char *lds, FdCount &cnt, bool &negeps)
{
    const int tid = threadIdx.x;
    // the range's tasks (as fd_range finds them)
    int k_ph = 0;
    while (k_ph + 1 < L.nph && b >= L.wg_end[k_ph]) ++k_ph;
    const int64_t bl = k_ph > 0 ? b - L.wg_end[k_ph - 1] : b;
    const int64_t tpw = L.tpw[k_ph], ntasks = L.ntasks[k_ph];
    const int64_t t0 = bl * tpw;
    const int R = (int)(t0 + tpw < ntasks ? tpw : ntasks - t0);
    const int64_t T0 = L.task_base[k_ph] + t0;
    int64_t cA = -1, cB = -1;
    if (tid < R) {
        const TaskCells tc = task_cells(P, T0 + tid);
        cA = tc.A;
        cB = tc.slot == 0 ? -1 : tc.B;
    }
    bool waited = false;
    auto wait = [&] {
        if (waited) return;
        waited = true;
        if (g > 0) {   // each wave polls the cells of its lanes' tasks
            bool ready = tid >= R;
            const uint64_t t_wait = wall_clock64();
            for (;;) {
                if (!ready) {
                    const uint32_t ea = __hip_atomic_load(epoch + cA, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
                    const uint32_t eb =
                        cB < 0 ? (uint32_t)g
                               : __hip_atomic_load(epoch + cB, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
                    ready = ea >= (uint32_t)g && eb >= (uint32_t)g;
                }
                if (__ballot(!ready) == 0ull) break;
                if (wall_clock64() - t_wait > kWaitTicks) {
                    if ((tid & 63) == 0) atomicOr(A.err, ERR_STALL);
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
        }
        // every wave has seen its cells released; no state access of the
        // range moves above the wait (the state loads are themselves
        // coherent, so no cache invalidation is needed)
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    fd_range<K, true>(P, L, b, lds, A, cnt, negeps, wait);
    // a range without pairs still orders its cells behind the predecessors
    wait();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);   // this wave's state stores have completed
    __syncthreads();                 // ... and those of the other waves
    if (tid < R) {
        __hip_atomic_store(epoch + cA, (uint32_t)g + 1u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        if (cB >= 0)
            __hip_atomic_store(epoch + cB, (uint32_t)g + 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

struct FdSweepArgs {
    const DevParams *Pp;
    const FdSweep *SW;
    const uint32_t *order;
    FdArgs A;
    uint32_t *work, *epoch;
    unsigned long long *counters;
};
// W: waves per SIMD the registers are held to (see FD_WIDE_MIN).
template <int K, int W>
__global__ __launch_bounds__(FD_THREADS, W) void k_fd_sweep(FdSweepArgs)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t s_item;
    const FdSweepArgs &a = kernel_argument<FdSweepArgs>();
    const int tid = threadIdx.x;
    FdCount cnt = {0u, 0u, 0u, 0u, 0u};
    bool negeps = false;
    for (;;) {
        const FdSweepArgs &b = reread(a);
        if (tid == 0) s_item = atomicAdd(b.work, 1u);
        __syncthreads();
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_item);
        const FdSweep &SW = reread(*b.SW);
        if (it >= SW.nitems) break;
        int g = 0;
        while (it >= SW.group_end[g]) ++g;
        // range index within group g
        fd_flow_range<K>(*b.Pp, SW.launch[g], g, b.order[it], b.A, b.epoch, lds, cnt, negeps);
    }
    const FdSweepArgs &b = reread(a);
    fd_flush_counters(cnt, negeps, b.counters, b.A.err);
}

// The one-launch sweep of many boxes (batched replicas, fused layout): the
// ranges of every box, group by group (all boxes' ranges of group 0, then of
// group 1, ...; a box's ranges of one group in its own order), handed out by
// one counter.  A range waits only on ranges of the previous group of its own
// box, all handed out before it, so the argument of the one-box sweep holds.
// While one box waits on its chain of groups the other boxes' ranges run.
struct FdBoxDesc {
    const DevParams *Pp;
    const FdSweep *SW;
    const uint32_t *order;
    FdArgs A;
    uint32_t *epoch;
    unsigned long long *counters;
};

// item_off[g * (nbox + 1) + b]: the first item of box b in group g; entry
// nbox of a row is the first item of the next group (nitems for the last)
template <int K>
__global__ __launch_bounds__(FD_THREADS) void k_fd_sweep_boxes(const FdBoxDesc *__restrict__ boxes,
                                                       const uint32_t *__restrict__ item_off,
                                                       int nbox, int ngroups, uint32_t nitems,
                                                       uint32_t *work)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ uint32_t s_item;
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s_item = atomicAdd(work, 1u);
        __syncthreads();
        const uint32_t it = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_item);
        if (it >= nitems) break;
        int g = 0;
        while (g + 1 < ngroups && it >= item_off[(int64_t)(g + 1) * (nbox + 1)]) ++g;
        const uint32_t *row = item_off + (int64_t)g * (nbox + 1);
        int lo = 0, hi = nbox;   // row[lo] <= it < row[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (it >= row[mid]) lo = mid;
            else hi = mid;
        }
        // box and group are the same in every lane: say so, so that the
        // descriptor and the box's parameters are read as scalars
        lo = __builtin_amdgcn_readfirstlane(lo);
        g = __builtin_amdgcn_readfirstlane(g);
        const FdBoxDesc &D = boxes[lo];
        const uint32_t gbeg = g > 0 ? D.SW->group_end[g - 1] : 0u;
        FdCount cnt = {0u, 0u, 0u, 0u, 0u};
        bool negeps = false;
        fd_flow_range<K>(*D.Pp, D.SW->launch[g], g, D.order[gbeg + (it - row[lo])], D.A, D.epoch,
                         lds, cnt, negeps);
        fd_flush_counters(cnt, negeps, D.counters, D.A.err);
    }
}

// ---------------------------------------------------------------- host side

namespace {

// class of a phase: 0 = own cell, else the number of non-zero components of
// its offset; parity set: the cell parities the phase touches
struct PhaseGeom {
    int cls;
    unsigned parity_set;
};

PhaseGeom phase_geom(int phase)
{
    PhaseGeom g;
    if (phase == 0) {
        g.cls = 0;
        g.parity_set = 0xFFu;
        return g;
    }
    const int o = (phase - 1) / 8, pi = (phase - 1) % 8, k = 14 + o;
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
    const int b = (dx & 1) | ((dy & 1) << 1) | ((dz & 1) << 2);
    g.cls = (dx != 0) + (dy != 0) + (dz != 0);
    g.parity_set = (1u << pi) | (1u << (pi ^ b));
    return g;
}

// per-task staging allowance at 17.5 particles per cell: mean participants
// and pair entries per task, and their spread (standard deviation per task),
// measured on jittered lattices; then a headroom factor on both capacities.
// The own-cell phase gains from room for the heavy ranges (lattice cells of
// 27 particles) while it stays under the LDS share of a workgroup at two
// waves per SIMD (20 KB on a 160 KB CU).
struct Allow {
    double mp, sp, me, se, room;
};
constexpr Allow kAllow[4] = {
    {17.5, 5.5, 143.0, 50.0, 1.25},   // own cell
    {26.2, 10.0, 102.0, 59.0, 1.0},   // face
    {14.7, 10.0, 25.2, 20.0, 1.0},    // edge
    {6.7, 5.0, 5.4, 4.5, 1.0},        // corner
};
// Tasks of one range: enough that the level steps of a batch hold many pairs ...
constexpr int kDefaultTasks[4] = {8, 8, 16, 24};
// ... unless a group then has fewer ranges than the GPU has slots to run them:
// below these ranges per group (own cell, face, edge, corner) a box is bound
// by the chain of 27 groups, which shorter ranges shorten (one-launch sweeps,
// ms, at 1 / 4 / 8 tasks: 0.61 / 0.65 / 0.70 for 32^3 particles, 1.23 / 0.74 /
// 0.79 for 48^3, 2.73 / 0.88 / 0.81 for 64^3).
constexpr int kGroupRanges[4] = {1700, 850, 600, 512};
// A sweep of at least FD_WIDE_MIN particles runs three waves per SIMD (168
// registers, 13.6 KB of LDS a workgroup), a smaller one two: its chain gains
// more from larger ranges (two against three waves, ms: 0.79 / 0.85 at 48^3,
// 0.83 / 0.90 at 64^3, 1.05 / 1.04 at 80^3, 1.90 / 1.81 at 2^20).
constexpr int64_t FD_WIDE_MIN = 400000;

int round_up(double x, int q)
{
    return (int)((std::ceil(x) + q - 1) / q) * q;
}

}  // namespace

void fd_class_caps(const sdpd_ctx *c, int k, int t, int &cp, int &ce)
{
    const double s = c->ncell > 0 ? ((double)c->n / (double)c->ncell) / 17.5 : 1.0;
    // within the LDS share of two waves per SIMD: boxes with dense cells
    // (small boxes have up to ~34 particles per cell) would otherwise take
    // tens of KB per workgroup and leave the CU a few workgroups
    const int lim = std::min(std::min(c->max_lds, 65536), c->lds_share);
    const double st = std::sqrt((double)t);
    const double room = kAllow[k].room;
    cp = round_up((t * kAllow[k].mp + 4.0 * st * kAllow[k].sp) * s * room, 16);
    ce = round_up((t * kAllow[k].me + 4.0 * st * kAllow[k].se) * s * s * room, 64);
    cp = std::min(std::max(cp, 128), 65535);
    ce = std::max(ce, 64);
    // shrink to the LDS limit, keeping the particle / pair proportion
    while (fd_lds_bytes(cp, ce) > (size_t)lim && (cp > 128 || ce > 64)) {
        cp = std::max(128, cp * 7 / 8);
        ce = std::max(64, ce * 7 / 8);
    }
}

// tasks per range t (about) of class k with the LDS capacities that go with it;
// a task of a box with dense cells has more pairs, as the density squared, and
// a range fewer tasks
static void fd_set_class(const sdpd_ctx *c, sdpd_tuning &u, int k, int t)
{
    const double s = c->ncell > 0 ? ((double)c->n / (double)c->ncell) / 17.5 : 1.0;
    if (s > 1.0) t = (int)std::lround(t / (s * s));
    t = std::min(std::max(t, 1), FD_MAXTASKS);
    int cp, ce;
    fd_class_caps(c, k, t, cp, ce);
    u.fd_tasks[k] = t;
    u.fd_lds_particles[k] = cp;
    u.fd_lds_pairs[k] = ce;
}

sdpd_tuning fd_batch_tuning(const sdpd_ctx *c, int64_t total)
{
    sdpd_tuning u;
    // many boxes share each launch, which ends with its slowest range: the
    // defaults, twice them where a launch holds several GPU-fulls of ranges
    // (ms per step at 8 / 16 tasks, cells of 17.5: 2.6 / 3.4 for 16 replica
    // boxes, 5.3 / 5.6 for 64, 18.0 / 16.6 for 192)
    for (int k = 0; k < 4; ++k)
        fd_set_class(c, u, k, kDefaultTasks[k] * (total > ((int64_t)1 << 21) ? 2 : 1));
    return u;
}

void fd_default_tuning(sdpd_ctx *c)
{
    c->fd_wide = c->n >= FD_WIDE_MIN;
    // LDS share of one workgroup at that many waves per SIMD
    c->lds_share = std::max(c->lds_cu / (c->fd_wide ? 12 : 8), 4096);
    for (int k = 0; k < 4; ++k) {
        const int64_t tasks = k == 0 ? c->ncell : c->ncell / 2;   // of a group of class k
        const int64_t fit = std::max<int64_t>(tasks / kGroupRanges[k], 1);
        fd_set_class(c, c->tuning, k, (int)std::min<int64_t>(kDefaultTasks[k], fit));
    }
    if (c->max_lds > 65536) {
        // allow dynamic LDS beyond 64 KiB where the device has it
        const void *kerns[] = {(const void *)k_fd_phase<0>, (const void *)k_fd_phase<1>,
                               (const void *)k_fd_phase<2>, (const void *)k_fd_sweep<0, 2>,
                               (const void *)k_fd_sweep<1, 2>, (const void *)k_fd_sweep<2, 2>,
                               (const void *)k_fd_sweep<0, 3>, (const void *)k_fd_sweep<1, 3>,
                               (const void *)k_fd_sweep<2, 3>,
                               (const void *)k_fd_records<0>, (const void *)k_fd_records<1>,
                               (const void *)k_fd_records<2>, (const void *)k_fd_levels<0>,
                               (const void *)k_fd_levels<1>, (const void *)k_fd_levels<2>,
                               (const void *)k_fd_phase_gen_multi,
                               (const void *)k_fd_phase_fast_multi,
                               (const void *)k_fd_phase_mix_multi};
        bool ok = true;
        for (const void *k : kerns)
            ok = ok && hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           c->max_lds) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            c->max_lds = 65536;
        }
    }
}

int fd_check_tuning(const sdpd_ctx *c, const sdpd_tuning *t)
{
    for (int k = 0; k < 4; ++k) {
        if (t->fd_tasks[k] < 1 || t->fd_tasks[k] > FD_MAXTASKS) return SDPD_EINVAL;
        if (t->fd_lds_particles[k] < 128 || t->fd_lds_particles[k] > 65535) return SDPD_EINVAL;
        if (t->fd_lds_pairs[k] < 64 || t->fd_lds_pairs[k] > (1 << 24)) return SDPD_EINVAL;
        if (fd_lds_checked_bytes(t->fd_lds_particles[k], t->fd_lds_pairs[k]) > (size_t)c->max_lds)
            return SDPD_EINVAL;
    }
    return SDPD_OK;
}

// the launches of a sweep: phase 0, then each phase gets the level 1 + the
// largest level of the earlier phases whose parity sets intersect its own,
// and the phases of one level run together (at most FD_MAXPH per launch)
static std::vector<std::vector<int>> fd_make_groups()
{
    std::vector<std::vector<int>> groups(1, std::vector<int>(1, 0));
    int lvl[105];
    unsigned set[105];
    int maxl = 0;
    for (int p = 1; p <= 104; ++p) {
        set[p] = phase_geom(p).parity_set;
        lvl[p] = 1;
        for (int r = 1; r < p; ++r)
            if ((set[r] & set[p]) && lvl[r] + 1 > lvl[p]) lvl[p] = lvl[r] + 1;
        maxl = std::max(maxl, lvl[p]);
    }
    for (int l = 1; l <= maxl; ++l) {
        std::vector<int> g;
        for (int p = 1; p <= 104; ++p) {
            if (lvl[p] != l) continue;
            g.push_back(p);
            if ((int)g.size() == FD_MAXPH) {
                groups.push_back(g);
                g.clear();
            }
        }
        if (!g.empty()) groups.push_back(g);
    }
    return groups;
}
static const std::vector<std::vector<int>> &fd_groups()   // (the same for every box)
{
    static const std::vector<std::vector<int>> groups = fd_make_groups();
    return groups;
}

// workgroup ranges that tuning u gives one launch over the tasks of up to
// FD_MAXPH mutually disjoint phases; returns the number of ranges
static int64_t fd_launch_geometry(const sdpd_ctx *c, const sdpd_tuning &u, const int *phases,
                                  int nph, FdLaunch &L)
{
    L.nph = nph;
    L.cap_p = 0;
    L.cap_e = 0;
    int64_t wg = 0;
    for (int k = 0; k < FD_MAXPH; ++k) {
        L.task_base[k] = L.ntasks[k] = L.wg_end[k] = 0;
        L.tpw[k] = 1;
    }
    for (int k = 0; k < nph; ++k) {
        const int ph = phases[k];
        const int cls = phase_geom(ph).cls;
        L.task_base[k] = ph == 0 ? 0 : c->ncell + (int64_t)(ph - 1) * (c->ncell / 8);
        L.ntasks[k] = ph == 0 ? c->ncell : c->ncell / 8;
        L.tpw[k] = u.fd_tasks[cls];
        wg += (L.ntasks[k] + L.tpw[k] - 1) / L.tpw[k];
        L.wg_end[k] = wg;
        L.cap_p = std::max(L.cap_p, (int)u.fd_lds_particles[cls]);
        L.cap_e = std::max(L.cap_e, (int)u.fd_lds_pairs[cls]);
    }
    return wg;
}

// The ranges of a whole sweep, group by group, that tuning u gives, and the LDS
// of a workgroup.  The epochs need every group to touch every cell exactly once:
// its phases' parity sets partition the 8 parities (true of the 26 groups of the
// 13 forward offsets; checked).
static int fd_sweep_ranges(const sdpd_ctx *c, const sdpd_tuning &u, FdSweep &h, size_t &lds)
{
    const std::vector<std::vector<int>> &groups = fd_groups();
    if ((int)groups.size() > FD_MAXGROUPS) return SDPD_EINVAL;
    memset(&h, 0, sizeof h);
    h.ngroups = (int)groups.size();
    int64_t total = 0;
    lds = 0;
    for (size_t g = 0; g < groups.size(); ++g) {
        unsigned cover = 0;
        for (int ph : groups[g]) {
            const unsigned ps = phase_geom(ph).parity_set;
            if (cover & ps) return SDPD_EINVAL;
            cover |= ps;
        }
        if (cover != 0xFFu) return SDPD_EINVAL;
        total += fd_launch_geometry(c, u, groups[g].data(), (int)groups[g].size(), h.launch[g]);
        if (total > 0x7fffffffLL) return SDPD_EINVAL;
        h.group_end[g] = (uint32_t)total;
        lds = std::max(lds, fd_lds_bytes(h.launch[g].cap_p, h.launch[g].cap_e));
    }
    h.nitems = (uint32_t)total;
    return lds > (size_t)c->max_lds ? SDPD_EINVAL : SDPD_OK;
}

// 16-byte units of the records of the largest batch of any range
static int64_t fd_record_slice(const FdSweep &h)
{
    int64_t ce = 1;
    for (int g = 0; g < h.ngroups; ++g) ce = std::max<int64_t>(ce, h.launch[g].cap_e);
    return 4 * ce;
}

static bool fd_fast(const sdpd_ctx *c)
{
    return c->dp.fd == SDPD_FD_EMS && c->dp.kernel == SDPD_KERNEL_LUCY && c->dp.par_twice_perp;
}

// kernel variant: 0 general, 1 the common case, 2 the common case with the
// FP32 proposal (mixed precision; other schemes keep the FP64 update)
static int fd_kind(const sdpd_ctx *c)
{
    return fd_fast(c) ? (c->dp.mixed ? 2 : 1) : 0;
}

using SweepKernel = void (*)(FdSweepArgs);
static SweepKernel fd_sweep_kernel(const sdpd_ctx *c)
{
    static const SweepKernel kern[2][3] = {{k_fd_sweep<0, 2>, k_fd_sweep<1, 2>, k_fd_sweep<2, 2>},
                                           {k_fd_sweep<0, 3>, k_fd_sweep<1, 3>, k_fd_sweep<2, 3>}};
    return kern[c->fd_wide][fd_kind(c)];
}

static FdArgs fd_args(const sdpd_ctx *c, const sdpd_state *s, double dt_fd)
{
    FdArgs A;
    A.qrho = reinterpret_cast<const double4 *>(c->q4);
    A.p = s->p;
    A.eps = s->eps;
    A.id = s->id;
    A.pair_off = c->pair_off;
    A.part_off = c->part_off;
    A.pairs = c->pairs;
    A.part_list = c->part_list;
    A.pair_cap = (uint32_t)c->pair_cap;
    A.part_cap = (uint32_t)c->part_cap;
    A.dstep = c->dstep;
    A.dt = dt_fd;
    A.y_c = -2.0 * dt_fd * c->dp.inv_m * c->dp.kperp_c * c->dp.cF;
    A.rec = reinterpret_cast<double2 *>(c->rec_buf);
    A.rec_stride = 0;
    A.lvl = c->lvl_end;
    A.err = c->err;
    return A;
}

bool fd_one_launch(const sdpd_ctx *c)
{
    if (c->fd_per_group || c->sweep_mode == SDPD_SWEEP_PER_GROUP) return false;
    return c->sweep_mode == SDPD_SWEEP_ONE || c->fd_dataflow;
}

// one launch per group
static int launch_phases(sdpd_ctx *c, const sdpd_state *s, const int *phases, int nph,
                         double dt_fd)
{
    FdLaunch L;
    const int64_t wg = fd_launch_geometry(c, c->tuning, phases, nph, L);
    if (wg == 0) return SDPD_OK;
    if (wg > 0x7fffffffLL) return SDPD_EINVAL;
    const size_t lds = fd_lds_bytes(L.cap_p, L.cap_e);
    if (lds > (size_t)c->max_lds) return SDPD_EINVAL;
    const FdPhaseArgs args{c->dparams, L, fd_args(c, s, dt_fd), c->counters};
    const int kind = fd_kind(c);
    const int rc =
        kind == 2 ? launch_or_record(c, k_fd_phase<2>, k_fd_phase_mix_multi, (unsigned)wg,
                                     FD_THREADS, lds, args)
        : kind == 1 ? launch_or_record(c, k_fd_phase<1>, k_fd_phase_fast_multi, (unsigned)wg,
                                       FD_THREADS, lds, args)
                    : launch_or_record(c, k_fd_phase<0>, k_fd_phase_gen_multi, (unsigned)wg,
                                       FD_THREADS, lds, args);
    return rc;
}

// The same with the records of the whole sweep formed first.  Both kernels cut
// the tasks into ranges and batches, and find the records and level ends by them:
// both take the ranges from the context's sweep table.
static int launch_records_and_levels(sdpd_ctx *c, const sdpd_state *s, double dt_fd)
{
    const FdSweep &h = *c->sweep_host;
    const FdArgs A = fd_args(c, s, dt_fd);
    const int kind = fd_kind(c);
    if (h.nitems == 0u) return SDPD_OK;
    auto records = kind == 2 ? k_fd_records<2> : kind == 1 ? k_fd_records<1> : k_fd_records<0>;
    hipLaunchKernelGGL(records, dim3(h.nitems), dim3(FD_THREADS), c->sweep_lds, c->stream,
                       c->dparams, (const FdSweep *)c->sweep, A);
    auto levels = kind == 2 ? k_fd_levels<2> : kind == 1 ? k_fd_levels<1> : k_fd_levels<0>;
    for (int g = 0; g < h.ngroups; ++g) {
        const FdLaunch &L = h.launch[g];
        const uint32_t wg = h.group_end[g] - (g > 0 ? h.group_end[g - 1] : 0u);
        if (wg == 0u) continue;
        hipLaunchKernelGGL(levels, dim3(wg), dim3(FD_THREADS), fd_lds_bytes(L.cap_p, L.cap_e),
                           c->stream, FdPhaseArgs{c->dparams, L, A, c->counters});
    }
    return check_hip(hipGetLastError());
}

// Order of the ranges inside each group: by the latest position, in the
// hand-out order, of the ranges of the previous group they wait for (ties in
// task order), so that ranges whose cells are released first are taken first.
// Every group touches every cell, so that position lies among those of the previous
// group: a counting sort.
static std::vector<uint32_t> fd_range_order(const sdpd_ctx *c, const FdSweep &h)
{
    const uint32_t nx = (uint32_t)c->dp.nc[0], ny = (uint32_t)c->dp.nc[1],
                   nz = (uint32_t)c->dp.nc[2], hx = nx / 2, hy = ny / 2;
    const uint32_t ncell = (uint32_t)c->ncell, per = ncell / 8;
    std::vector<uint32_t> order(h.nitems);
    std::vector<uint32_t> last(ncell, 0u);   // hand-out position of the range that last touched a cell
    std::vector<uint32_t> key, at, cells;    // cells: of the group's ranges, one after the other
    std::vector<size_t> cells_end;
    uint32_t before = 0, begin = 0;          // first position of the previous group and of this one
    for (int g = 0; g < h.ngroups; ++g) {
        const FdLaunch &L = h.launch[g];
        const uint32_t nb = h.group_end[g] - begin;
        key.assign(nb, before);
        cells.clear();
        cells_end.resize(nb);
        uint32_t b = 0;
        for (int k_ph = 0; k_ph < L.nph; ++k_ph) {
            // the phase's tasks (as task_cells numbers them): A of parity pi, B = A + delta_o
            const bool own = L.task_base[k_ph] == 0;
            const uint32_t ph = own ? 0u : (uint32_t)(L.task_base[k_ph] - ncell) / per;
            const uint32_t pi = ph % 8u, k = 14u + ph / 8u;
            const uint32_t dx = k % 3u + nx - 1u, dy = (k / 3u) % 3u + ny - 1u, dz = k / 9u + nz - 1u;
            uint32_t tx = 0, ty = 0, tz = 0;
            for (int64_t t0 = 0; t0 < L.ntasks[k_ph]; t0 += L.tpw[k_ph], ++b) {
                const int64_t t1 = std::min(t0 + L.tpw[k_ph], L.ntasks[k_ph]);
                for (int64_t t = t0; t < t1; ++t) {
                    if (own) {
                        cells.push_back((uint32_t)t);
                        continue;
                    }
                    const uint32_t ax = 2u * tx + (pi & 1u), ay = 2u * ty + ((pi >> 1) & 1u),
                                   az = 2u * tz + (pi >> 2);
                    const uint32_t A = ax + nx * (ay + ny * az);
                    const uint32_t B = (ax + dx) % nx + nx * ((ay + dy) % ny + ny * ((az + dz) % nz));
                    cells.push_back(A);
                    cells.push_back(B);
                    key[b] = std::max(key[b], std::max(last[A], last[B]));
                    if (++tx == hx) {
                        tx = 0;
                        if (++ty == hy) {
                            ty = 0;
                            ++tz;
                        }
                    }
                }
                cells_end[b] = cells.size();
            }
        }
        at.assign((size_t)(begin - before) + 2u, 0u);   // ranges of each key, then their places
        for (uint32_t r = 0; r < nb; ++r) ++at[key[r] - before + 1u];
        for (size_t x = 1; x < at.size(); ++x) at[x] += at[x - 1];
        for (uint32_t r = 0; r < nb; ++r) {
            const uint32_t place = begin + at[key[r] - before]++;
            order[place] = r;
            for (size_t x = r ? cells_end[r - 1] : 0; x < cells_end[r]; ++x) last[cells[x]] = place;
        }
        before = begin;
        begin = h.group_end[g];
    }
    return order;
}

// Layout of the sweep that SDPD_SWEEP_AUTO takes for the ranges h.
// One launch when the sweep holds at least three GPU-fulls of ranges (at
// two waves per SIMD; boxes of some 450 cells); a smaller one mostly waits
// on its chain of 27 groups, and one launch per group then holds no
// workgroup slots while it waits.  Where the process asks for more queues than
// the default four, boxes on many streams would hold them against each other
// (256 boxes of 13^3 to 40^3 particles stepped eagerly on 32 streams and queues:
// 312 ms per step with the line above, 88 with one launch per group; 48 boxes on
// four streams and queues: 23 and 25): there only boxes that fill the GPU by
// themselves, four GPU-fulls of ranges of full size (some 7,900 cells; one box
// alone with eight queues, one launch / one per group, ms: 0.95 / 1.34 at 48^3
// particles, 1.21 / 1.57 at 56^3, 3.04 / 4.41 at 2^20).
static int fd_auto_layout(sdpd_ctx *c, const FdSweep &h)
{
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) !=
            hipSuccess || cus < 1) {
        (void)hipGetLastError();
        return SDPD_EHIP;
    }
    const int64_t full = 8 * (int64_t)cus;
    c->fd_dataflow = (int64_t)h.nitems >= 3 * full;
    if (!c->fd_dataflow || hw_queues() <= 4) return SDPD_OK;
    FdSweep large = h;
    if (c->tune_gen == 0) {   // (the defaults of smaller boxes are shorter ranges)
        sdpd_tuning u = c->tuning;
        for (int k = 0; k < 4; ++k) u.fd_tasks[k] = std::max(u.fd_tasks[k], kDefaultTasks[k]);
        size_t lds = 0;
        const int rc = fd_sweep_ranges(c, u, large, lds);
        if (rc) return rc;
    }
    c->fd_dataflow = (int64_t)large.nitems >= 4 * full;
    return SDPD_OK;
}

// workgroups of the one-launch sweep over the ranges h: as many as run at once
static int fd_sweep_grid(const sdpd_ctx *c, const FdSweep &h, size_t lds, int &grid)
{
    int per_cu = 0, cus = 0;
    const void *kern = (const void *)fd_sweep_kernel(c);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, FD_THREADS, lds) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) !=
            hipSuccess || per_cu < 1 || cus < 1) {
        (void)hipGetLastError();
        return SDPD_EHIP;
    }
    grid = (int)std::min<int64_t>((int64_t)per_cu * cus, std::max<int64_t>(h.nitems, 1));
    return SDPD_OK;
}

int fd_choose_layout(sdpd_ctx *c, size_t &slices)
{
    FdSweep h;
    size_t lds = 0;
    int grid = 0;
    int rc = fd_sweep_ranges(c, c->tuning, h, lds);
    if (!rc) rc = fd_auto_layout(c, h);
    if (!rc) rc = fd_sweep_grid(c, h, lds, grid);
    slices = sizeof(double2) * (size_t)fd_record_slice(h) * (size_t)grid;
    return rc;
}

// The records of one group of the sweep, for launches per group: 2 KB per particle, which
// a box swept by one launch only takes when it is first asked for another layout.
int fd_group_records(sdpd_ctx *c)
{
    if (c->rec_buf || c->prm.fd == SDPD_FD_NONE || c->n == 0) return SDPD_OK;
    const size_t bytes = fd_group_record_bytes(c);
    if (hipMalloc(&c->rec_own, bytes) != hipSuccess) {
        c->rec_own = nullptr;
        (void)hipGetLastError();
        return SDPD_ENOMEM;
    }
    c->rec_buf = static_cast<double *>(c->rec_own);
    c->rec_bytes = bytes;
    return SDPD_OK;
}

// Record slices of the one-launch sweep's workgroups: in the context's workspace (its
// slices, or its records of a group) when they fit, else in a buffer of their own.
static int fd_flow_records(sdpd_ctx *c, const FdSweep &h)
{
    if (c->prm.fd == SDPD_FD_NONE || c->n == 0) return SDPD_OK;
    c->sweep_rec_stride = fd_record_slice(h);
    const size_t need = sizeof(double2) * (size_t)c->sweep_rec_stride * (size_t)c->sweep_grid;
    double *const held = need <= c->slice_bytes ? c->slices : need <= c->rec_bytes ? c->rec_buf
                                                                                   : nullptr;
    if (c->flow_own && (held || c->flow_own_bytes < need)) {
        (void)hipFree(c->flow_own);
        c->flow_own = nullptr;
        c->flow_own_bytes = 0;
    }
    if (!held && !c->flow_own) {
        if (hipMalloc(&c->flow_own, need) != hipSuccess) {
            c->flow_own = nullptr;
            (void)hipGetLastError();
            return SDPD_ENOMEM;
        }
        c->flow_own_bytes = need;
    }
    c->flow_rec = held ? held : static_cast<double *>(c->flow_own);
    return SDPD_OK;
}

// Table of the sweep kernel (ranges of every group, in sweep order) and its
// launch size, rebuilt whenever the tuning changes.
int fd_prepare_sweep(sdpd_ctx *c)
{
    // the table and the order are rewritten in place: no sweep may be running
    if (hipStreamSynchronize(c->stream) != hipSuccess) return SDPD_EHIP;
    c->sweep_ok = 0;
    auto table = std::make_shared<FdSweep>();
    FdSweep &h = *table;
    size_t lds = 0;
    int rc = fd_sweep_ranges(c, c->tuning, h, lds);
    if (rc) return rc;
    c->sweep_host = table;
    if (!c->sweep && hipMalloc(&c->sweep, sizeof(FdSweep)) != hipSuccess) {
        c->sweep = nullptr;
        (void)hipGetLastError();
        return SDPD_ENOMEM;
    }
    if ((rc = check_hip(hipMemcpy(c->sweep, &h, sizeof h, hipMemcpyHostToDevice)))) return rc;
    const std::vector<uint32_t> order = fd_range_order(c, h);
    // one range per task at most: the buffer is sized once and never moves
    const size_t order_cap = (size_t)NMASK * (size_t)c->ncell + 1;
    if (order.size() > order_cap) return SDPD_EINVAL;
    if (!c->sweep_order &&
        hipMalloc((void **)&c->sweep_order, sizeof(uint32_t) * order_cap) != hipSuccess) {
        c->sweep_order = nullptr;
        (void)hipGetLastError();
        return SDPD_ENOMEM;
    }
    if (!order.empty() &&
        (rc = check_hip(hipMemcpy(c->sweep_order, order.data(), sizeof(uint32_t) * order.size(),
                                  hipMemcpyHostToDevice))))
        return rc;
    if ((rc = fd_sweep_grid(c, h, lds, c->sweep_grid))) return rc;
    c->sweep_lds = lds;
    if ((rc = fd_flow_records(c, h))) return rc;
    if ((rc = fd_auto_layout(c, h))) return rc;
    if (!fd_one_launch(c) && (rc = fd_group_records(c))) return rc;
    c->sweep_ok = 1;
    return SDPD_OK;
}

// (x, y, z, rho) record of every particle for the pair gathers of the sweep
struct PackArgs {
    int64_t n;
    const double *q, *rho;
    double4 *qrho;
};
__device__ __forceinline__ void pack_qrho_body(const PackArgs &a, uint32_t blk)
{
    const int64_t n = a.n;
    const double *__restrict__ q = a.q;
    const double *__restrict__ rho = a.rho;
    double4 *qrho = a.qrho;
    const int64_t i = (int64_t)blk * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double4 r;
    r.x = q[i];
    r.y = q[n + i];
    r.z = q[2 * n + i];
    r.w = rho[i];
    qrho[i] = r;
}
__global__ void k_pack_qrho(PackArgs a) { pack_qrho_body(a, blockIdx.x); }
SDPD_MULTI_KERNEL(k_pack_qrho_multi, PackArgs, pack_qrho_body, 256)

// Schedule and packed records of a sweep (independent of the tuning), then
// its launches.
int fd_sweep_prepare(sdpd_ctx *c, const sdpd_state *s, bool packed)
{
    int rc = run_schedule(c);
    if (rc) return rc;
    if (!packed) {
        timer_begin(c, TK_SCHED);   // sweep preparation, with the schedule
        rc = launch_or_record(c, k_pack_qrho, k_pack_qrho_multi, (unsigned)((c->n + 255) / 256),
                              256, 0,
                              PackArgs{c->n, s->q, s->rho, reinterpret_cast<double4 *>(c->q4)});
        timer_end(c, TK_SCHED);
        if (rc) return rc;
    }
    c->fd_swept = 1;
    return SDPD_OK;
}

int fd_launch_sweep(sdpd_ctx *c, const sdpd_state *s, double dt_fd)
{
    if (!c->sweep_ok) return SDPD_EINVAL;
    int rc;
    const int kind = fd_kind(c);
    if (c->rec && c->fd_record_flow) {
        // fused batch: the epochs start at zero, then the sweep is recorded
        // as this box's part of one multi-box launch
        if ((rc = launch_fill_u32(c, c->epoch, 0u, c->ncell))) return rc;
        FdBoxDesc d;
        d.Pp = c->dparams;
        d.SW = (const FdSweep *)c->sweep;
        d.order = c->sweep_order;
        d.A = fd_args(c, s, dt_fd);
        d.epoch = c->epoch;
        d.counters = c->counters;
        RecordedLaunch r;
        r.multi = nullptr;
        r.grid = 1;
        r.block = FD_THREADS;
        r.lds = c->sweep_lds;
        r.flow_kind = kind;
        r.args.resize(sizeof d);
        memcpy(r.args.data(), &d, sizeof d);
        c->rec->push_back(std::move(r));
        return SDPD_OK;
    }
    if (!fd_one_launch(c)) {
        if (!c->rec_buf) return SDPD_ENOMEM;   // (made with the layout)
        // records of the whole sweep first, where the context holds them all
        // (a small box on its own; recorded launches share the GPU with other
        // boxes, where forming the records in the launches is faster)
        const bool whole = c->lvl_end && !c->rec && !c->fd_per_group;
        timer_begin(c, TK_FD);
        if (whole) {
            if ((rc = launch_records_and_levels(c, s, dt_fd))) return rc;
        } else {
            for (const std::vector<int> &g : fd_groups())
                if ((rc = launch_phases(c, s, g.data(), (int)g.size(), dt_fd))) return rc;
        }
        timer_end(c, TK_FD);
        return SDPD_OK;
    }
    // epochs of the cells and the range counter start at zero
    if ((rc = launch_fill_u32(c, c->epoch, 0u, c->ncell + 1))) return rc;
    timer_begin(c, TK_FD);
    FdArgs A = fd_args(c, s, dt_fd);
    A.rec = reinterpret_cast<double2 *>(c->flow_rec);
    A.rec_stride = c->sweep_rec_stride;
    hipLaunchKernelGGL(fd_sweep_kernel(c), dim3((unsigned)c->sweep_grid), dim3(FD_THREADS), c->sweep_lds, c->stream,
                       FdSweepArgs{c->dparams, (const FdSweep *)c->sweep, c->sweep_order, A,
                                   c->epoch + c->ncell, c->epoch, c->counters});
    timer_end(c, TK_FD);
    return check_hip(hipGetLastError());
}

// A box's ranges in a launch shared with other boxes (`total` particles in all): those
// of its batch tuning, with table and order in buffers of the launch's own, or of the
// box's own tuning where its user has set one (a later change invalidates the batch).
static int fd_flow_tables(sdpd_ctx *c, int64_t total, FdBoxDesc &d, size_t &lds, FdSweep &h,
                          FlowSweep &out)
{
    const bool own = c->tune_gen == 0;
    int rc = fd_sweep_ranges(c, own ? fd_batch_tuning(c, total) : c->tuning, h, lds);
    if (rc || !own) return rc;
    const std::vector<uint32_t> order = fd_range_order(c, h);
    const size_t bytes[2] = {sizeof h, sizeof(uint32_t) * order.size()};
    const void *src[2] = {&h, order.data()};
    void *dst[2] = {nullptr, nullptr};
    for (int k = 0; k < 2; ++k) {
        if (hipMalloc(&dst[k], bytes[k] ? bytes[k] : 4) != hipSuccess) return SDPD_ENOMEM;
        out.tables.push_back(dst[k]);
        if (bytes[k] && (rc = check_hip(hipMemcpy(dst[k], src[k], bytes[k], hipMemcpyHostToDevice))))
            return rc;
    }
    d.SW = (const FdSweep *)dst[0];
    d.order = (const uint32_t *)dst[1];
    return SDPD_OK;
}

int fd_flow_build(const std::vector<sdpd_ctx *> &ctxs,
                  const std::vector<const RecordedLaunch *> &recs, FlowSweep &out)
{
    const int nbox = (int)ctxs.size();
    if (nbox < 1 || recs.size() != ctxs.size()) return SDPD_EINVAL;
    out.kind = recs[0]->flow_kind;
    out.nbox = nbox;
    out.ngroups = ctxs[0]->sweep_host ? ctxs[0]->sweep_host->ngroups : 0;
    std::vector<FdBoxDesc> desc(nbox);
    std::vector<uint32_t> ends((size_t)nbox * FD_MAXGROUPS);
    out.lds = 0;
    int64_t stride = 0, total = 0;   // record slice of a workgroup: the largest of any box
    for (sdpd_ctx *c : ctxs) total += c->n;
    for (int b = 0; b < nbox; ++b) {
        if (recs[b]->flow_kind != out.kind || recs[b]->args.size() != sizeof(FdBoxDesc))
            return SDPD_EINVAL;
        memcpy(&desc[b], recs[b]->args.data(), sizeof(FdBoxDesc));
        size_t lds = 0;
        FdSweep h;
        const int rc = fd_flow_tables(ctxs[b], total, desc[b], lds, h, out);
        if (rc) return rc;
        if (h.ngroups != out.ngroups) return SDPD_EINVAL;
        memcpy(&ends[(size_t)b * FD_MAXGROUPS], h.group_end, sizeof h.group_end);
        out.lds = std::max(out.lds, lds);
        stride = std::max(stride, fd_record_slice(h));
    }
    // group-major item numbering: all boxes' ranges of group 0, then group 1, ...
    std::vector<uint32_t> off((size_t)out.ngroups * (nbox + 1));
    uint64_t item = 0;
    for (int g = 0; g < out.ngroups; ++g)
        for (int b = 0; b <= nbox; ++b) {
            off[(size_t)g * (nbox + 1) + b] = (uint32_t)item;
            if (b < nbox) {
                const uint32_t *ge = &ends[(size_t)b * FD_MAXGROUPS];
                item += ge[g] - (g > 0 ? ge[g - 1] : 0u);
                if (item > 0x7fffffffull) return SDPD_EINVAL;
            }
        }
    out.nitems = (uint32_t)item;
    int per_cu = 0, cus = 0;
    const void *kern = out.kind == 2 ? (const void *)k_fd_sweep_boxes<2>
                       : out.kind == 1 ? (const void *)k_fd_sweep_boxes<1>
                                       : (const void *)k_fd_sweep_boxes<0>;
    if (out.lds > 65536 &&
        hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)out.lds) !=
            hipSuccess)
        return SDPD_EINVAL;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, FD_THREADS, out.lds) !=
            hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctxs[0]->device) !=
            hipSuccess || per_cu < 1 || cus < 1) {
        (void)hipGetLastError();
        return SDPD_EHIP;
    }
    out.grid = (unsigned)std::min<int64_t>((int64_t)per_cu * cus, std::max<int64_t>(item, 1));
    if (hipMalloc((void **)&out.rec, sizeof(double2) * (size_t)stride * out.grid) != hipSuccess)
        return SDPD_ENOMEM;
    for (FdBoxDesc &d : desc) {
        d.A.rec = reinterpret_cast<double2 *>(out.rec);
        d.A.rec_stride = stride;
    }
    if (hipMalloc(&out.boxes, sizeof(FdBoxDesc) * nbox) != hipSuccess ||
        hipMalloc((void **)&out.item_off, sizeof(uint32_t) * off.size()) != hipSuccess ||
        hipMalloc((void **)&out.work, sizeof(uint32_t)) != hipSuccess)
        return SDPD_ENOMEM;
    int rc = check_hip(hipMemcpy(out.boxes, desc.data(), sizeof(FdBoxDesc) * nbox,
                                 hipMemcpyHostToDevice));
    if (!rc)
        rc = check_hip(hipMemcpy(out.item_off, off.data(), sizeof(uint32_t) * off.size(),
                                 hipMemcpyHostToDevice));
    return rc;
}

// counter of the multi-box sweep back to zero (a kernel, so that a captured
// graph holds no memset node)
__global__ void k_flow_reset(uint32_t *work)
{
    if (threadIdx.x == 0) *work = 0u;
}

int fd_flow_launch(const FlowSweep &f, hipStream_t stream)
{
    if (f.nitems == 0) return SDPD_OK;
    hipLaunchKernelGGL(k_flow_reset, dim3(1), dim3(64), 0, stream, f.work);
    const FdBoxDesc *boxes = (const FdBoxDesc *)f.boxes;
    if (f.kind == 2)
        hipLaunchKernelGGL(k_fd_sweep_boxes<2>, dim3(f.grid), dim3(FD_THREADS), f.lds, stream,
                           boxes, f.item_off, f.nbox, f.ngroups, f.nitems, f.work);
    else if (f.kind == 1)
        hipLaunchKernelGGL(k_fd_sweep_boxes<1>, dim3(f.grid), dim3(FD_THREADS), f.lds, stream,
                           boxes, f.item_off, f.nbox, f.ngroups, f.nitems, f.work);
    else
        hipLaunchKernelGGL(k_fd_sweep_boxes<0>, dim3(f.grid), dim3(FD_THREADS), f.lds, stream,
                           boxes, f.item_off, f.nbox, f.ngroups, f.nitems, f.work);
    return check_hip(hipGetLastError());
}

void fd_flow_free(FlowSweep &f)
{
    if (f.boxes) (void)hipFree(f.boxes);
    if (f.item_off) (void)hipFree(f.item_off);
    if (f.work) (void)hipFree(f.work);
    if (f.rec) (void)hipFree(f.rec);
    f.rec = nullptr;
    for (void *t : f.tables) (void)hipFree(t);
    f.tables.clear();
    f.boxes = nullptr;
    f.item_off = nullptr;
    f.work = nullptr;
}

// The step index of the draws is read from c->dstep on the device (set by
// the caller, or advanced inside a captured graph).
int run_fd_sweep(sdpd_ctx *c, const sdpd_state *s, double dt_fd, bool packed)
{
    if (c->prm.fd == SDPD_FD_NONE || c->n == 0) return SDPD_OK;
    const int rc = fd_sweep_prepare(c, s, packed);
    return rc ? rc : fd_launch_sweep(c, s, dt_fd);
}

}  // namespace sdpd
