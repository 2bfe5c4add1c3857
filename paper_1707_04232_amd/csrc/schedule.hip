// Pair schedule of the fluctuation/dissipation sweep, built once per sweep
// from the active-pair masks of the density pass.
//
// Tasks are numbered in sweep order: phase 0 holds one task per cell A
// (pairs inside A); phase 1 + 8 o + pi holds one task per cell A of
// coordinate parity pi (pairs between A and A + delta_o), in the order
// tx + hx (ty + hy tz) of A = 2 (tx, ty, tz) + parity bits.  For every task
// this pass writes, contiguously in task order,
//   * the list of particles that take part in one of its pairs: the A-cell
//     ones by slot, then (inter-cell tasks) the B-cell ones by slot;
//   * its active pairs in round order (round = slot_A XOR slot_B, the
//     order that defines the sweep), each with its level: 1 + the largest
//     level among the earlier pairs of the task that share a particle.
//     Pairs of equal level in one task share no particle.
// Pair entry (64 bits): the phase-relative list positions of its two
// particles (25 bits each) and the level (bits 50..56).
#include <type_traits>

#include "fd_math.hpp"
#include "tasks.hpp"

namespace sdpd {

// pairs and participating particles of every task: one 16-lane quarter-wave
// per task (a cell holds 16 particles on average), lane x reading the masks
// of slots x, x + 16, ... of cell A, then sums and ORs over the quarter
// (all mask loads of a task in flight at once)
constexpr int COUNT_WAVES = 4;     // waves per workgroup
constexpr int COUNT_LANES = 16;    // lanes per task: four tasks per wave

struct TaskCountArgs {
    const DevParams *Pp;
    const uint32_t *cell_start;
    const uint64_t *masks;
    uint32_t *tcount, *tnp;
};
__device__ __forceinline__ void task_count_body(const TaskCountArgs &a, uint32_t blk)
{
    const DevParams &P = *a.Pp;
    const uint32_t *__restrict__ cell_start = a.cell_start;
    const uint64_t *__restrict__ masks = a.masks;
    uint32_t *tcount = a.tcount, *tnp = a.tnp;
    const int lane = threadIdx.x & 63, x = lane & (COUNT_LANES - 1);
    const int64_t T = ((int64_t)blk * COUNT_WAVES + (threadIdx.x >> 6)) * (64 / COUNT_LANES) +
                      lane / COUNT_LANES;
    const bool ok = T < (int64_t)NMASK * P.ncell;
    uint32_t c = 0, na = 0;
    uint64_t orb = 0;
    int slot = 0;
    if (ok) {
        const TaskCells tc = task_cells(P, T);
        slot = tc.slot;
        const uint32_t sA = cell_start[tc.A], nA = cell_start[tc.A + 1] - sA;
        const uint32_t nB = cell_start[tc.B + 1] - cell_start[tc.B];
        if (nA <= (uint32_t)P.cap && nB <= (uint32_t)P.cap) {
            for (uint32_t a = (uint32_t)x; a < nA; a += COUNT_LANES) {
                const uint64_t m = masks[(int64_t)tc.slot * P.n + sA + a];
                na += m != 0ull;
                orb |= m;
                c += (uint32_t)__popcll(tc.slot == 0 ? (m & ~((2ull << a) - 1ull)) : m);
            }
        }
    }
#pragma unroll
    for (int off = COUNT_LANES / 2; off > 0; off >>= 1) {   // stays inside the quarter
        c += (uint32_t)__shfl_xor((int)c, off);
        na += (uint32_t)__shfl_xor((int)na, off);
        orb |= (uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)orb, off) |
               ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(orb >> 32), off) << 32);
    }
    if (ok && x == 0) {
        tcount[T] = c;
        tnp[T] = na + (slot == 0 ? 0u : (uint32_t)__popcll(orb));
    }
}
__global__ __launch_bounds__(64 * COUNT_WAVES) void k_task_count(TaskCountArgs a)
{
    task_count_body(a, xcd_block(blockIdx.x, gridDim.x));
}
SDPD_MULTI_KERNEL(k_task_count_multi, TaskCountArgs, task_count_body, 64 * COUNT_WAVES)

struct TaskSpan {
    TaskCells tc;
    uint32_t sA, nA, sB, nB, e0, e1, q0, q1, rel;
};

__device__ __forceinline__ TaskSpan task_span(const DevParams &P, const uint32_t *cell_start,
                                              const uint32_t *pair_off, const uint32_t *part_off,
                                              int64_t T)
{
    TaskSpan t;
    t.tc = task_cells(P, T);
    t.sA = cell_start[t.tc.A];
    t.nA = cell_start[t.tc.A + 1] - t.sA;
    t.sB = cell_start[t.tc.B];
    t.nB = cell_start[t.tc.B + 1] - t.sB;
    t.e0 = pair_off[T];
    t.e1 = pair_off[T + 1];
    t.q0 = part_off[T];
    t.q1 = part_off[T + 1];
    t.rel = t.q0 - part_off[phase_base(P.ncell, t.tc.phase)];
    return t;
}

// OR over the lanes of one W-lane segment
template <int W>
__device__ __forceinline__ uint64_t seg_or64(uint64_t v)
{
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int off = W / 2; off > 0; off >>= 1) {
        lo |= (uint32_t)__shfl_xor((int)lo, off);
        hi |= (uint32_t)__shfl_xor((int)hi, off);
    }
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// One task on a W-lane segment of the wave (W = 64: the whole wave; W = 32:
// one half, for cells of at most 32 particles, so that every slot and every
// round partner x ^ s lies in the half).  Lane x of the segment is slot x of
// cell A and of cell B.  Writes the task's particle list and its pairs in
// round order with their levels.  `ok` = this segment has a task to do;
// INTRA (a phase-0 task) is the same for the whole wave (tasks of one pair
// never mix phase 0 with the others, since ncell is even).
template <int W, bool INTRA>
__device__ __forceinline__ void schedule_segment(const DevParams &P, const TaskSpan &t, bool ok,
                                                 const uint64_t *__restrict__ masks,
                                                 uint64_t *pairs, uint32_t *part_list)
{
    constexpr bool intra = INTRA;
    using M = typename std::conditional<W == 32, uint32_t, uint64_t>::type;
    const int lane = threadIdx.x & 63;
    const int base = lane & ~(W - 1), x = lane & (W - 1);
    const bool hi = base != 0;
    const M below = (M)(((uint64_t)1 << x) - 1u);   // x < W <= 64
    const uint64_t mask64 = ok && (uint32_t)x < t.nA
                                ? masks[(int64_t)t.tc.slot * P.n + t.sA + x] : 0ull;
    const M mask = (M)mask64;   // W = 32: partner slots < 32
    const uint64_t bact = __ballot(mask != 0);
    const M actA = (M)(hi ? (bact >> 32) : bact);
    const M actB = intra ? actA : (M)seg_or64<W>(mask);
    const uint32_t nactA = (uint32_t)__popcll(actA);
    // particle list: A-side participants by slot, then (inter-cell) B-side
    if ((actA >> x) & 1u) part_list[t.q0 + __popcll(actA & below)] = t.sA + (uint32_t)x;
    if (!intra && ((actB >> x) & 1u))
        part_list[t.q0 + nactA + __popcll(actB & below)] = t.sB + (uint32_t)x;
    // phase-relative list positions of this lane as A-side and as B-side particle
    const uint32_t posA = t.rel + (uint32_t)__popcll(actA & below);
    const uint32_t posB = intra ? posA : t.rel + nactA + (uint32_t)__popcll(actB & below);
    const M rm = (M)xor_permute_bits(mask, (uint32_t)x);   // bit s: partner x ^ s active
    uint64_t r = seg_or64<W>(rm);
    if (W == 32) r |= (uint32_t)__shfl_xor((int)(uint32_t)r, 32);   // union of the halves
    uint64_t rounds = uniform64(r);
    int LA = 0, LB = 0;
    uint32_t pos = t.e0;
    while (rounds) {
        const int s = __builtin_ctzll(rounds);   // uniform
        rounds &= rounds - 1;
        const int partner = x ^ s;                // < W
        const int addr = (base + partner) << 2;   // byte address of the partner lane
        const bool act = (rm >> s) & 1u;
        const int la = __builtin_amdgcn_ds_bpermute(addr, LA);
        const uint32_t pB = (uint32_t)__builtin_amdgcn_ds_bpermute(addr, (int)posB);
        bool own;
        if (INTRA) {   // one role per particle; the pair's two lanes agree on act
            own = act && x < partner;
            LA = act ? max(LA, la) + 1 : LA;
        } else {       // lane x is slot x of cell A and slot x of cell B
            const int lb = __builtin_amdgcn_ds_bpermute(addr, LB);
            const bool actB_here = __builtin_amdgcn_ds_bpermute(addr, (int)act) != 0;
            own = act;
            const int nLA = act ? max(LA, lb) + 1 : LA;
            LB = actB_here ? max(LB, la) + 1 : LB;
            LA = nLA;
        }
        const uint64_t bal = __ballot(own);
        const uint32_t blo = (uint32_t)bal, bhi = (uint32_t)(bal >> 32);
        if (own) {
            // rank among the owning lanes of this segment
            uint32_t k = __builtin_amdgcn_mbcnt_hi(bhi, __builtin_amdgcn_mbcnt_lo(blo, 0u));
            if (W == 32 && hi) k -= (uint32_t)__popc(blo);
            const uint64_t e = (uint64_t)posA | ((uint64_t)pB << 25) | ((uint64_t)LA << 50);
            pairs[pos + k] = e;
        }
        pos += W == 32 ? (uint32_t)__popc(hi ? bhi : blo) : (uint32_t)__popcll(bal);
    }
}

// levels, particle lists and pair entries (grid-stride over pairs of
// consecutive tasks; 14 * ncell is even).  Both tasks of a pair run side by
// side in the two halves of the wave when all their cells hold at most 32
// particles, otherwise one after the other on the whole wave.
constexpr int SCHED_WAVES = 4;   // waves per workgroup, each on its own task pairs

struct ScheduleArgs {
    const DevParams *Pp;
    const uint32_t *cell_start;
    const uint64_t *masks;
    const uint32_t *pair_off, *part_off;
    uint64_t *pairs;
    uint32_t *part_list;
    uint32_t pair_cap, part_cap;
    uint32_t *err;
    uint32_t nblk;   // workgroups of the box's grid-stride loop
};
__device__ __forceinline__ void schedule_body(const ScheduleArgs &a, uint32_t blk)
{
    const DevParams &P = *a.Pp;
    const uint32_t *__restrict__ cell_start = a.cell_start;
    const uint64_t *__restrict__ masks = a.masks;
    const uint32_t *__restrict__ pair_off = a.pair_off;
    const uint32_t *__restrict__ part_off = a.part_off;
    uint64_t *pairs = a.pairs;
    uint32_t *part_list = a.part_list;
    const uint32_t pair_cap = a.pair_cap, part_cap = a.part_cap;
    uint32_t *err = a.err;
    const int64_t ntask = (int64_t)NMASK * P.ncell;
    // wave index made explicitly uniform: the task arithmetic below then runs
    // on the scalar unit once per wave
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    for (int64_t Wp = (int64_t)blk * SCHED_WAVES + wave; 2 * Wp < ntask;
         Wp += (int64_t)a.nblk * SCHED_WAVES) {
        const TaskSpan ta = task_span(P, cell_start, pair_off, part_off, 2 * Wp);
        const TaskSpan tb = task_span(P, cell_start, pair_off, part_off, 2 * Wp + 1);
        bool oka = ta.e1 > ta.e0, okb = tb.e1 > tb.e0;
        const bool bada = oka && (ta.nA > (uint32_t)P.cap || ta.nB > (uint32_t)P.cap ||
                                  ta.e1 > pair_cap || ta.q1 > part_cap);
        const bool badb = okb && (tb.nA > (uint32_t)P.cap || tb.nB > (uint32_t)P.cap ||
                                  tb.e1 > pair_cap || tb.q1 > part_cap);
        if (bada || badb) {
            if (lane == 0) atomicOr(err, ERR_PAIRCAP);
            oka = oka && !bada;
            okb = okb && !badb;
        }
        if (!oka && !okb) continue;
        uint32_t widest = 0;
        if (oka) widest = max(ta.nA, ta.nB);
        if (okb) widest = max(widest, max(tb.nA, tb.nB));
        if (widest <= 32) {
            const bool hi = lane >= 32;
            const TaskSpan t = hi ? tb : ta;   // field-wise select
            if (ta.tc.slot == 0)   // both tasks of the pair are of one kind
                schedule_segment<32, true>(P, t, hi ? okb : oka, masks, pairs, part_list);
            else
                schedule_segment<32, false>(P, t, hi ? okb : oka, masks, pairs, part_list);
        } else {
            if (oka) {
                if (ta.tc.slot == 0) schedule_segment<64, true>(P, ta, true, masks, pairs, part_list);
                else schedule_segment<64, false>(P, ta, true, masks, pairs, part_list);
            }
            if (okb) {
                if (tb.tc.slot == 0) schedule_segment<64, true>(P, tb, true, masks, pairs, part_list);
                else schedule_segment<64, false>(P, tb, true, masks, pairs, part_list);
            }
        }
    }
}

__global__ __launch_bounds__(64 * SCHED_WAVES) void k_schedule(ScheduleArgs a)
{
    schedule_body(a, xcd_block(blockIdx.x, gridDim.x));
}
SDPD_MULTI_KERNEL(k_schedule_multi, ScheduleArgs, schedule_body, 64 * SCHED_WAVES)

// ---------------------------------------------------------------- large boxes
// The same lists with the serial part at full lane occupancy: a wave takes 64
// consecutive tasks.  Part 1, two tasks at a time with lane x on slot x (as
// schedule_segment<32>): the participants, the particle list, and for every round s
// the word of the slots x of cell A whose partner x ^ s is active, by a bit
// transpose over the lanes.  Part 2, one lane per task: the pairs in round order
// (words in ascending s, bits in ascending x), each level from the levels of its two
// slots in LDS.  Entries leave through LDS, eight per task and store.  Tasks with a
// cell of more than 32 particles run on the whole wave as schedule_segment<64>.
//
// schedule_segment runs one round of two tasks at a time, with two of its 64 lanes
// in use on average: bound by the VALU at 335 instructions per particle.  This one
// takes 90 and is bound by LDS latency at ten waves per CU (their words): 1M
// particles 520 -> 240 us, 8M 4.1 -> 1.75 ms.  Two pairs per step of part 2, the
// next word read ahead without a branch and the masks read before the first store
// (a load waits for the stores before it) are worth a third of that.
constexpr int SCHED_TASKS = 64;        // tasks per wave
constexpr int SCHED_TASK_WAVES = 1;    // waves per workgroup (14.6 KB of LDS)
constexpr int SCHED_CHUNK = 8;         // entries of a task per store
constexpr int SCHED_LV = 68;           // bytes of a lane's levels (32 + 32, padded)

struct ScheduleLds {
    uint32_t word[33 * SCHED_TASKS];   // word s of task t at [64 s + ((t + s) & 63)]; 32: zeros
    uint8_t level[SCHED_LV * SCHED_TASKS];
    uint32_t stage[(SCHED_CHUNK + 1) * SCHED_TASKS];   // entry u of task t at [9 t + u]
};

__device__ __forceinline__ void sched_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)   // J < 32
{
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, J << 10 | 0x1f);
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// bit b of m to bit b ^ x
template <int SH>
__device__ __forceinline__ uint32_t xor_step(uint32_t m, uint32_t x, uint32_t low)
{
    const uint32_t sw = ((m & low) << SH) | ((m >> SH) & low);
    return x & (uint32_t)SH ? sw : m;
}
__device__ __forceinline__ uint32_t xor_permute32(uint32_t m, uint32_t x)
{
    m = xor_step<1>(m, x, 0x55555555u);
    m = xor_step<2>(m, x, 0x33333333u);
    m = xor_step<4>(m, x, 0x0f0f0f0fu);
    m = xor_step<8>(m, x, 0x00ff00ffu);
    return x & 16u ? __builtin_amdgcn_alignbit(m, m, 16) : m;
}

// 32 x 32 bits over the 32 lanes of each half: bit s of lane x to bit x of lane s
template <int J>
__device__ __forceinline__ uint32_t transpose_step(uint32_t v, uint32_t x, uint32_t low)
{
    const uint32_t t = lane_xor<J>(v);
    const bool up = (x & (uint32_t)J) != 0u;
    const uint32_t keep = up ? ~low : low;                       // columns that stay
    const uint32_t moved = __builtin_amdgcn_alignbit(t, t, up ? J : 32 - J);
    return (v & keep) | (moved & ~keep);
}
__device__ __forceinline__ uint32_t transpose32(uint32_t v, uint32_t x)
{
    v = transpose_step<16>(v, x, 0x0000ffffu);
    v = transpose_step<8>(v, x, 0x00ff00ffu);
    v = transpose_step<4>(v, x, 0x0f0f0f0fu);
    v = transpose_step<2>(v, x, 0x33333333u);
    return transpose_step<1>(v, x, 0x55555555u);
}

__device__ __forceinline__ void schedule_tasks(const ScheduleArgs &a, int64_t T0, ScheduleLds &lds)
{
    const DevParams &P = *a.Pp;
    const int lane = threadIdx.x & 63;
    const int64_t n = P.n, ntask = (int64_t)NMASK * P.ncell, T = T0 + lane;
    const uint32_t *__restrict__ words = reinterpret_cast<const uint32_t *>(a.masks);
    const bool in = T < ntask;
    const TaskSpan t = task_span(P, a.cell_start, a.pair_off, a.part_off, in ? T : ntask - 1);
    bool ok = in && t.e1 > t.e0;
    if (ok && (t.nA > (uint32_t)P.cap || t.nB > (uint32_t)P.cap || t.e1 > a.pair_cap ||
               t.q1 > a.part_cap)) {
        atomicOr(a.err, ERR_PAIRCAP);
        ok = false;
    }
    const bool wide = ok && max(t.nA, t.nB) > 32u;
    for (uint64_t big = __ballot(wide); big; big &= big - 1ull) {
        const TaskSpan u =
            task_span(P, a.cell_start, a.pair_off, a.part_off, T0 + __builtin_ctzll(big));
        if (u.tc.slot == 0) schedule_segment<64, true>(P, u, true, a.masks, a.pairs, a.part_list);
        else schedule_segment<64, false>(P, u, true, a.masks, a.pairs, a.part_list);
    }
    ok = ok && !wide;
    const uint64_t todo = __ballot(ok);
    if (!todo) return;

    // part 1
    uint32_t actA = 0u, actB = 0u, rounds = 0u;   // of this lane's task
    const int x = lane & 31, half = lane >> 5;
    const uint32_t below = (1u << x) - 1u;
    // The masks go to LDS first, each to where its lane's word will be: between the
    // stores of the lists every load would have to wait for the stores before it.
    constexpr int U = 8, ITS = SCHED_TASKS / 2;
    const uint32_t n_a = ok ? t.nA : 0u;
    auto place = [&](int it) { return 64 * x + ((2 * it + half + x) & 63); };
    for (int it0 = 0; it0 < ITS; it0 += U) {
        uint32_t v[U], live[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int it = it0 + u, src = 2 * it + half;
            const uint32_t sA = (uint32_t)__shfl((int)t.sA, src);
            live[u] = (uint32_t)x < (uint32_t)__shfl((int)n_a, src);
            const int slot = __builtin_amdgcn_readlane(t.tc.slot, 2 * it);   // of both
            // the index, 0 past the last slot, without a branch around the load
            uint64_t at = (uint64_t)slot * (uint64_t)n + sA + (uint32_t)x;
            at = live[u] ? at : 0ull;
            asm volatile("" : "+v"(at));
            v[u] = words[2 * at];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) lds.word[place(it0 + u)] = live[u] ? v[u] : 0u;
    }
    for (int it0 = 0; it0 < ITS; it0 += 4) {
        if (((todo >> (2 * it0)) & 255ull) == 0ull) continue;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int src = 2 * (it0 + u) + half;
            const uint32_t sA = (uint32_t)__shfl((int)t.sA, src);
            const uint32_t sB = (uint32_t)__shfl((int)t.sB, src);
            const uint32_t q0 = (uint32_t)__shfl((int)t.q0, src);
            const uint32_t m = lds.word[place(it0 + u)];
            const int it = it0 + u;
            const bool intra = __builtin_amdgcn_readlane(t.tc.slot, 2 * it) == 0;
            const uint64_t ba = __ballot(m != 0u);
            const uint32_t aA = half ? (uint32_t)(ba >> 32) : (uint32_t)ba;
            uint32_t aB = m;
            aB |= lane_xor<1>(aB);
            aB |= lane_xor<2>(aB);
            aB |= lane_xor<4>(aB);
            aB |= lane_xor<8>(aB);
            aB |= lane_xor<16>(aB);
            if (intra) aB = aA;
            // a pair inside a cell belongs to its lower slot
            const uint32_t own = intra ? m & ~below & ~(1u << x) : m;
            const uint32_t w = transpose32(xor_permute32(own, (uint32_t)x), (uint32_t)x);
            lds.word[place(it)] = w;
            if ((aA >> x) & 1u) a.part_list[q0 + __popc(aA & below)] = sA + (uint32_t)x;
            if (!intra && ((aB >> x) & 1u))
                a.part_list[q0 + __popc(aA) + __popc(aB & below)] = sB + (uint32_t)x;
            const uint64_t br = __ballot(w != 0u);
            const uint32_t bB0 = lane_value(aB, 0), bB1 = lane_value(aB, 32);
            if (lane >> 1 == it) {
                const bool odd = lane & 1;
                actA = odd ? (uint32_t)(ba >> 32) : (uint32_t)ba;
                rounds = odd ? (uint32_t)(br >> 32) : (uint32_t)br;
                actB = odd ? bB1 : bB0;
            }
        }
    }
    // part 2
    uint8_t *const lvA = lds.level + SCHED_LV * lane;
    uint8_t *const lvB = t.tc.slot == 0 ? lvA : lvA + 32;
    for (int b = 0; b < 64; b += 4) *reinterpret_cast<uint32_t *>(lvA + b) = 0u;
    lds.word[64 * 32 + lane] = 0u;
    sched_sync();
    const uint32_t first_b = t.tc.slot == 0 ? 0u : (uint32_t)__popc(actA);
    auto word = [&](uint32_t s) { return lds.word[64u * s + (((uint32_t)lane + s) & 63u)]; };
    // the word in work, and the next one (past the last: word 32), read ahead
    uint32_t cur = 0u, s = 0u, s_nxt = rounds ? (uint32_t)__builtin_ctz(rounds) : 32u;
    uint32_t nxt = word(s_nxt);
    rounds &= rounds - 1u;
    uint32_t *const stage = lds.stage + (SCHED_CHUNK + 1) * lane;
    uint32_t e = t.e0;
    while (__any((cur | nxt) != 0u)) {
        uint32_t made = 0u;
        for (int it = 0; it < SCHED_CHUNK / 2; ++it) {
            const bool step = cur == 0u;
            cur = step ? nxt : cur;
            s = step ? s_nxt : s;
            const uint32_t ahead = rounds ? (uint32_t)__builtin_ctz(rounds) : 32u;
            s_nxt = step ? ahead : s_nxt;
            rounds = step ? rounds & (rounds - 1u) : rounds;
            nxt = word(s_nxt);
            if (cur) {
                // two pairs of the round at once (they share no particle); of one
                // pair only, the second does the same again
                const uint32_t rest = cur & (cur - 1u);
                const uint32_t xa[2] = {(uint32_t)__builtin_ctz(cur),
                                        (uint32_t)__builtin_ctz(rest ? rest : cur)};
                cur = rest & (rest - 1u);
                uint32_t level[2];
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    level[u] = max((uint32_t)lvA[xa[u]], (uint32_t)lvB[xa[u] ^ s]) + 1u;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t xb = xa[u] ^ s;
                    lvA[xa[u]] = lvB[xb] = (uint8_t)level[u];
                    const uint32_t pa = (uint32_t)__popc(actA & ((1u << xa[u]) - 1u));
                    const uint32_t pb = first_b + (uint32_t)__popc(actB & ((1u << xb) - 1u));
                    stage[made + (uint32_t)u] = pa | pb << 8 | level[u] << 16;
                }
                made += rest ? 2u : 1u;
            }
        }
        sched_sync();
        const int u = lane & (SCHED_CHUNK - 1);
#pragma unroll
        for (int r = 0; r < SCHED_TASKS; r += 64 / SCHED_CHUNK) {
            const int src = r + lane / SCHED_CHUNK;
            const uint32_t cnt = (uint32_t)__shfl((int)made, src);
            const uint32_t at = (uint32_t)__shfl((int)e, src) + (uint32_t)u;
            const uint64_t rel = (uint64_t)(uint32_t)__shfl((int)t.rel, src);
            const uint64_t v = lds.stage[(SCHED_CHUNK + 1) * src + u];
            if ((uint32_t)u < cnt)
                a.pairs[at] = (rel + (v & 255u)) | (rel + ((v >> 8) & 255u)) << 25 |
                              (v >> 16) << 50;
        }
        e += made;
        sched_sync();
    }
}
__device__ __forceinline__ void schedule_tasks_body(const ScheduleArgs &a, uint32_t blk)
{
    __shared__ ScheduleLds lds[SCHED_TASK_WAVES];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t T0 = ((int64_t)blk * SCHED_TASK_WAVES + wave) * SCHED_TASKS;
    if (T0 < (int64_t)NMASK * a.Pp->ncell) schedule_tasks(a, T0, lds[wave]);
}
__global__ __launch_bounds__(64 * SCHED_TASK_WAVES) void k_schedule_tasks(ScheduleArgs a)
{
    schedule_tasks_body(a, xcd_block(blockIdx.x, gridDim.x));
}
SDPD_MULTI_KERNEL(k_schedule_tasks_multi, ScheduleArgs, schedule_tasks_body,
                  64 * SCHED_TASK_WAVES)

// With fewer cells a lane's pairs one after the other take longer than they save:
// counts, scans and schedule of 1728 cells 46 us (tasks on lanes: 88), 7128 cells
// 109 (102), 13824 cells 162 (130), 61250 cells 600 (336).  In launches recorded for
// a batch the cells of all boxes that share the launch count (64 boxes of 1000 to
// 17000 particles, two steps: 8.87 -> 8.69 ms).
constexpr int64_t SCHED_TASKS_MIN_CELLS = 6 << 10;

int run_schedule(sdpd_ctx *c)
{
    const int64_t ntask = (int64_t)NMASK * c->ncell;
    timer_begin(c, TK_SCHED);
    const int64_t per_block = (int64_t)COUNT_WAVES * (64 / COUNT_LANES);
    const int64_t count_blocks = (ntask + per_block - 1) / per_block;
    int rc = launch_or_record(c, k_task_count, k_task_count_multi, (unsigned)count_blocks,
                              64 * COUNT_WAVES, 0,
                              TaskCountArgs{c->dparams, c->cell_start, c->masks, c->task_count,
                                            c->task_np});
    if (rc) return rc;
    if ((rc = run_scan(c, c->task_count, c->pair_off, c->task_np, c->part_off, ntask,
                       c->block_sums, -1, false)))
        return rc;
    // one workgroup per pair of tasks: many independent short waves hide the
    // load latency
    const int64_t grid = std::min<int64_t>((ntask / 2 + SCHED_WAVES - 1) / SCHED_WAVES, 0x7fffffffLL);
    const ScheduleArgs args{c->dparams, c->cell_start, c->masks, c->pair_off, c->part_off,
                            c->pairs, c->part_list, (uint32_t)c->pair_cap, (uint32_t)c->part_cap,
                            c->err, (uint32_t)grid};
    if (std::max(c->ncell, c->batch_cells) >= SCHED_TASKS_MIN_CELLS) {
        const int64_t per = (int64_t)SCHED_TASK_WAVES * SCHED_TASKS;
        rc = launch_or_record(c, k_schedule_tasks, k_schedule_tasks_multi,
                              (unsigned)((ntask + per - 1) / per), 64 * SCHED_TASK_WAVES, 0,
                              args);
    } else {
        rc = launch_or_record(c, k_schedule, k_schedule_multi, (unsigned)grid, 64 * SCHED_WAVES,
                              0, args);
    }
    timer_end(c, TK_SCHED);
    return rc;
}

}  // namespace sdpd
