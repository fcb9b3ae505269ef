// Descending sweep of graphs whose tensors are numbered as they are created (operator after operator, no gaps) and
// whose operators read recent tensors or graph inputs only -- recorded graphs that are long and thin.
//
// A tensor's consumers all have larger operator ids than its producer.  A workgroup of W waves walks one graph's
// operators from the highest id down, 64 W at a time, and keeps M of the tensors around the place it has reached in
// a ring in LDS: every input edge of the group falls into the ring or on a graph input, and M of the graph inputs
// lives in LDS for the whole sweep.  So no push ever goes to memory, nothing is hashed, and no output of the walk
// depends on a load of M: what is read from memory is the adjacency, once, and what is written is every word of M
// and K, once, in runs of consecutive words.  Target bits are kept in registers (packed tensor and set) and dropped into
// the ring when it comes to cover their tensor; nothing has to be cleared or seeded before the kernel starts.
//
// Dependencies inside a group: every lane ORs M of its operator's outputs, pushes the bits it had not seen into the
// ring slots of those inputs that the group itself writes, and looks again until no lane sees a new bit; all other
// inputs get their bits once, when the group is final.  A wave settles on its own first (LDS operations of a wave
// complete in order, so that needs no barrier); barriers pass the bits on between waves, one more round for every hop
// that crosses from one wave to another.
//
// What a graph must satisfy is found out when it is built (k_records_and_check): operators in topological order,
// outputs in one run up to the graph's last tensor, at most `low` graph inputs, no input further than `dist` below the
// end of its operator's own outputs, at most `span64` outputs per 64 operators.  The ring holds dist + 3 W span64 tensors,
// rounded up to a power of two: the group, everything it reads, and two groups of slack, so that a target bit may arrive
// one group late.
//
// More than 64 sets of a single graph are words of 64 that have nothing to do with each other: a workgroup each.  150 sets
// on a graph of 20 000 operators, one word after the other before: 0.84 ms -> 0.30.
//
// Segments.  Where no operator reads further back than 64 tensors, a graph is cut into segments of a few words that are swept
// at the same time, a wave each (eight, or one, put its targets in place before).  What a segment lacks is M of the 64 tensors at
// its upper boundary, and everything in it is an OR of what its own targets give and of some of those 64: so it is swept twice, once
// with the targets that lie in it, once with the 64 tensors as 64 sets, whose masks then say which of them reach what.  k_ring_join works out M of the boundaries
// from the top down and adds what they bring; in a batch k_ring_carry has done so before, per graph, and counted.
// Which graphs, how long and what it measured: ring_segments in api.hip.
//
// What bounds it.  One wave per graph and few graphs: the chain of LDS round trips, 270 cycles per settling step and
// 4.4 steps per 64 operators whose inputs are drawn from the last 64 tensors (2 900 cycles per 64 operators in all; the hash
// tables of k_sweep_graphs took 19 000).  4 096 graphs: the memory, 37 bytes per operator.  Measured on graphs of that
// family, 64 sets, whole prune: 4 096 graphs of 20 000 operators 3.13 -> 1.18 ms, 96 of 3 001 0.49 -> 0.094, one of 20 000
// 3.3 -> 0.28 (level by level before), one of 2 000 0.21 -> 0.052; in segments the last three 0.054, 0.050 and 0.035: launches and
// the wait 14 us, the sweep 10 to 18 (6 before the first operator, 1 per word), the boundaries and the list 9 to 17.
#include <type_traits>

#include "common.h"

namespace dgn {

// Per-set counts without a transpose per group: every lane counts, for its own operators, how often each of the 64
// bits was set, in bit-sliced form (plane i holds bit i of all 64 counters).  Four masks are folded at a time with
// full adders; only the resulting carry of weight 4 ripples through the higher planes.
constexpr int kRingPlanes = 13;                     // counters up to 2^13 - 1 words of 64 operators per wave
static_assert(kRingMaxGraphOps / kWave < (1 << kRingPlanes), "a single wave counts all words of the largest graph");

struct RingCount {
    u64 plane[kRingPlanes];
    u64 x0, x1, x2;                                 // masks waiting for the fourth
};

__device__ __forceinline__ void ring_add(u64 a, u64 b, u64 c, u64 &sum, u64 &carry)
{
    const u64 ab = a ^ b;
    sum = ab ^ c;
    carry = (ab & c) | (a & b);
}

__device__ __forceinline__ void ring_fold(RingCount &c, u64 x3, int planes_used)
{
    u64 s, ca, cb, cc;
    ring_add(c.plane[0], c.x0, c.x1, s, ca);
    ring_add(s, c.x2, x3, c.plane[0], cb);
    ring_add(c.plane[1], ca, cb, c.plane[1], cc);
#pragma unroll
    for (int i = 2; i < kRingPlanes; ++i) {
        if (i < planes_used) {                      // wave-uniform
            const u64 t = c.plane[i] & cc;
            c.plane[i] ^= cc;
            cc = t;
        }
    }
}

// LDS words by their address: what a lane keeps for a slot is the operand of the LDS instruction itself
typedef __attribute__((address_space(3))) u64 LdsWord;
__device__ __forceinline__ LdsWord *lds_word(uint32_t addr) { return (LdsWord *)(uintptr_t)addr; }
__device__ __forceinline__ u64 lds_read(uint32_t addr)
{
    return __hip_atomic_load(lds_word(addr), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_write(uint32_t addr, u64 v)
{
    __hip_atomic_store(lds_word(addr), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_or(uint32_t addr, u64 v)
{
    (void)__hip_atomic_fetch_or(lds_word(addr), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// What a lane knows of its operator before its turn comes.  Everything is fetched without a branch (lanes without an
// operator, and inputs past the end of a row, read some neighbour's instead), so that the number of loads in flight is
// known and a wait for one of them does not become a wait for all.  Offsets are 32-bit byte offsets from uniform bases.
struct RingRow {
    int ob, oe, ib, ie;                             // rows in out_idx / in_idx
    int32_t t[4];                                   // its first four inputs
};

template <typename T> __device__ __forceinline__ T &at_byte(T *base, uint32_t off)
{
    return *reinterpret_cast<T *>(reinterpret_cast<char *>(const_cast<std::remove_const_t<T> *>(base)) + off);
}

// in_row / out_row: the row pointers of the graph's n operators; i: operator within the graph
__device__ __forceinline__ void ring_bounds(const int32_t *in_row, const int32_t *out_row, RingRow &r, int i, int n)
{
    const uint32_t off = (uint32_t)min(max(i, 0), n - 1) * 4u;
    r.ob = at_byte(out_row, off);
    r.oe = at_byte(out_row, off + 4);
    r.ib = at_byte(in_row, off);
    r.ie = at_byte(in_row, off + 4);
}

__device__ __forceinline__ void ring_targets(const GraphView &g, RingRow &r)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) r.t[j] = at_byte(g.in_idx, (uint32_t)min(r.ib + j, g.nnz_in - 1) * 4u);
}

__device__ __forceinline__ void wave_fence()                 // LDS accesses of a wave complete in order: for the compiler alone
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A zero that the compiler takes for a value of its own in every lane: added to an address that is the same in all lanes,
// it keeps the load's result in a vector register until it is used (moved to a scalar one at once, as it would be, the
// wave would wait for the load where it is issued).
__device__ __forceinline__ uint32_t lane_zero()
{
    uint32_t z;
    asm("v_mov_b32 %0, 0" : "=v"(z));
    return z;
}

// What the last workgroup's thread leaves: the header for recycling, and the status for the host.  st: as in RingArgs::graphs.
__device__ __forceinline__ void ring_finish(const RingArgs &a, int4 st)
{
    // (member by member: copied whole, it would pass through scratch memory in every thread)
    a.hdr->magic = a.recycle && !st.y ? a.want.magic : 0;
    a.hdr->graph_serial = a.want.graph_serial;
    a.hdr->M = a.want.M;
    a.hdr->K = a.want.K;
    a.hdr->kept_ops = a.want.kept_ops;
    a.hdr->kept_count = a.want.kept_count;
    a.hdr->flags = a.want.flags;
    a.hdr->also_M = a.want.also_M;
    a.hdr->also_K = a.want.also_K;
    a.host_status[0] = st.y;
    a.host_status[1] = st.z;
    a.host_status[2] = st.w;
}

// W waves sweep.  H = 0: whole graphs; else a segment of one (W = 1), whose targets H waves put in place before.
template <int W, int H>
__global__ __launch_bounds__((H > W ? H : W) * kWave) void k_ring_sweep(RingArgs a)
{
    constexpr bool kSeg = H > 0;
    static_assert(!kSeg || W == 1, "a wave per segment");
    constexpr int N = W * kWave, kPlace = (H > W ? H : W) * kWave;         // threads that sweep, and that put the targets in place
    // [R] ring, [low] graph inputs, [1] a word that stays zero, [64] words that take what goes nowhere; targets; with the
    // list made here: running counts per word
    extern __shared__ u64 ring[];
    __shared__ int s_flag[3];                       // "a push crossed waves", by round
    __shared__ int s_total[W];                      // kept operators of each wave's word
    __shared__ int s_err, s_relax;
    __shared__ int s_lowest, s_own;                 // segments: the lowest target and how many
    __shared__ int32_t s_row[kWave + 1];            // the graph's target row pointers
    const GraphView &g = a.g;
    const int lane = lane_id(), wave = W > 1 ? (int)(threadIdx.x >> 6) : 0, tid = threadIdx.x;
    const bool batched = g.num_graphs > 1;
    // graph of a batch, or word of 64 sets; segments: a graph, a segment of it, a word of sets, of which the last is the boundary's
    const int gi = batched || kSeg ? blockIdx.x : 0, wd = kSeg ? blockIdx.z : batched ? 0 : blockIdx.x;
    const int seg = kSeg ? blockIdx.y : 0;
    const bool boundary = kSeg && wd == a.words;
    const int num_sets = min(a.num_sets - wd * kWave, kWave);
    const int64_t set0 = batched ? (int64_t)gi * num_sets : (int64_t)wd * kWave;    // first set of this workgroup
    const int64_t g_lo = batched ? g.op_off[gi] : 0;
    const int n_all = (int)((batched ? g.op_off[gi + 1] : g.num_ops) - g_lo);
    const int first = kSeg ? min(seg * a.seg_words * kWave, n_all) : 0, n = kSeg ? min(n_all - first, a.seg_words * kWave) : n_all;
    if (kSeg && (seg > 0 || boundary) && (n == 0 || (boundary && first + n == n_all))) return;      // (nothing comes in at the top)
    const int64_t o_lo = g_lo + first;
    const int32_t t_lo = batched ? (int32_t)g.t_off[gi] : 0, t_end = batched ? (int32_t)g.t_off[gi + 1] : g.num_tensors;
    const int32_t *in_row = g.in_rowptr + o_lo, *out_row = g.out_rowptr + o_lo;
    u64 *all_M = boundary ? a.b_M : a.M + (int64_t)wd * g.num_tensors;
    u64 *M = all_M + t_lo, *K = (boundary ? a.b_K : a.K + (int64_t)wd * g.num_ops) + o_lo;
    uint8_t *flags = !kSeg && a.flags ? a.flags + (int64_t)wd * g.num_ops + o_lo : nullptr;
    // outputs end with the graph's last tensor: output edge e is tensor e + shift; tensors below t_first are graph inputs
    const int32_t shift = t_end - (kSeg ? g.out_rowptr[g_lo + n_all] : out_row[n]);
    const int32_t t_first = (kSeg ? g.out_rowptr[g_lo] : out_row[0]) + shift;
    // the tensors that these operators write (the whole graph: all but its inputs)
    const int32_t t_hi = kSeg ? out_row[n] + shift : t_end, t_mine = kSeg ? out_row[0] + shift : t_first;
    // LDS: tensor t sits in the ring at slot t mod R, R a power of two, or among the inputs at t - t_lo
    const int R = a.ring_words;
    const uint32_t base = (uint32_t)(uintptr_t)(LdsWord *)ring;
    const uint32_t low_at = base + (uint32_t)(R - t_lo) * 8u, zero_at = base + (uint32_t)(R + a.low_words) * 8u;
    const uint32_t nowhere = zero_at + 8u + (uint32_t)lane * 8u;
    uint32_t *seeds = reinterpret_cast<uint32_t *>(ring + R + a.low_words + 1 + kWave);
    int *s_cum = reinterpret_cast<int *>(seeds + a.seed_words);
    auto slot_of = [&](int32_t t) { return base + (uint32_t)(t & (R - 1)) * 8u; };
    auto low_of = [&](int32_t t) { return low_at + (uint32_t)t * 8u; };
    static_assert(kRingExtraWords == 1 + kWave, "words behind the inputs");
    const bool found = a.recycle && same_header(*a.hdr, a.want);      // words that were zero need not be written again
    const bool skips = found && !kSeg;
    // what the first groups of operators need is on its way while the targets are put in place (not where a wave sweeps a whole
    // graph, of thousands: it takes longer with all of them asking at once)
    const int n_words = (n + kWave - 1) >> 6;
    const int steps = (n_words + W - 1) / W;
    int word = n_words - 1 - wave;                           // this wave's word of 64 operators
    int32_t z_next = 0;                                      // first output row of a group, as loaded
    const uint32_t vz = lane_zero();
    RingRow cur{}, nxt{}, nxt2{};
    auto group_first = [&](int step) { return (uint32_t)max((n_words - (step + 1) * W) * kWave, 0); };   // first operator
    auto first_bounds = [&]() {
        if (steps == 0) return;
        ring_bounds(in_row, out_row, cur, word * kWave + lane, n);
        ring_bounds(in_row, out_row, nxt, (word - W) * kWave + lane, n);
        if (W > 1) z_next = at_byte(out_row, group_first(0) * 4u + vz);
    };
    if (W > 1 || (kSeg && tid < N)) first_bounds();
    for (int i = tid; i <= R + a.low_words; i += kPlace) ring[i] = 0;
    if (tid < 3) s_flag[tid] = 0;
    if (tid == 0) s_err = s_relax = 0;
    if (kSeg && tid == 0) {
        s_own = 0;
        s_lowest = 0x7fffffff;
    }

    // the graph's targets, packed: tensor relative to t_lo in the upper 26 bits, set in the lower 6
    if (!boundary)
        for (int q = tid; q <= num_sets; q += kPlace) s_row[q] = a.tgt_rowptr[set0 + q];
    __syncthreads();
    const int64_t j0 = boundary ? 0 : max(s_row[0], 0), j1 = boundary ? 0 : min((int64_t)s_row[num_sets], a.num_targets);
    const bool from_m = j1 - j0 > a.seed_words || t_end - t_lo >= (1 << 26);         // too many: by way of M itself
    if (from_m) {
        if (kSeg && seg == 0)
            for (int64_t t = tid; t < t_first - t_lo; t += kPlace) store_coherent(&M[t], (u64)0);
        for (int64_t t = (kSeg ? t_mine - t_lo : 0) + tid; t < t_hi - t_lo; t += kPlace) store_coherent(&M[t], (u64)0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    }
    __syncthreads();
    int err = 0, lowest = 0x7fffffff;               // lowest: smallest target of this thread, relative to t_lo
    if constexpr (kSeg) {
        // Every segment looks at all of its graph's targets and keeps its own.  Its one wave takes 0.35 us for 64 of them (0.8 with a
        // branch for every one), so that where few workgroups run there are more waves for this than for the sweep.  Rows of 64
        // four at a time, their loads and searches side by side and without branches.
        auto look = [&](auto rows, int64_t first_j) {
            constexpr int kRows = decltype(rows)::value;
            int32_t t[kRows], j[kRows], lo[kRows];
#pragma unroll
            for (int c = 0; c < kRows; ++c) {
                j[c] = (int32_t)min(first_j + c * kWave + lane, j1 - 1);
                t[c] = a.tgt_idx[j[c]];
                lo[c] = 0;
            }
#pragma unroll
            for (int half = kWave / 2; half > 0; half >>= 1) {
                if (half >= num_sets) continue;              // uniform
                int32_t row[kRows];
#pragma unroll
                for (int c = 0; c < kRows; ++c) row[c] = s_row[min(lo[c] + half, num_sets)];
#pragma unroll
                for (int c = 0; c < kRows; ++c) lo[c] += lo[c] + half < num_sets && row[c] <= j[c] ? half : 0;
            }
            int32_t begin[kRows], end[kRows];
#pragma unroll
            for (int c = 0; c < kRows; ++c) {
                begin[c] = s_row[lo[c]];
                end[c] = s_row[lo[c] + 1];
            }
#pragma unroll
            for (int c = 0; c < kRows; ++c) {
                const bool is = first_j + c * kWave + lane < j1 && begin[c] <= j[c] && j[c] < end[c];      // (else it belongs to no set)
                const bool inside = t[c] >= t_lo && t[c] < t_end;
                if (is && !inside) err |= t[c] < 0 || t[c] >= g.num_tensors ? kErrIdRange : kErrCrossGraph;
                const bool low = is && inside && t[c] < t_first && seg == 0, mine = is && t[c] >= t_mine && t[c] < t_hi;
                if (from_m) {
                    if (low || mine) (void)atomicOr(&all_M[t[c]], (u64)1 << lo[c]);
                    continue;
                }
                if (low) lds_or(low_of(t[c]), (u64)1 << lo[c]);
                const u64 which = ballot64(mine);
                if (which == 0) continue;
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_own, __popcll(which));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(which & lanemask_lt());
                if (mine) {
                    lowest = min(lowest, t[c] - t_lo);
                    seeds[at] = ((uint32_t)(t[c] - t_lo) << 6) | (uint32_t)lo[c];
                }
            }
        };
        constexpr int kRows = 4;
        for (int64_t first_j = j0 + (tid & ~(kWave - 1)) * kRows; first_j < j1; first_j += kRows * kPlace) {
            if (j1 - first_j <= kWave) look(std::integral_constant<int, 1>{}, first_j);
            else look(std::integral_constant<int, kRows>{}, first_j);
        }
    } else {
        for (int64_t j = j0 + tid; j < j1; j += N) {
            uint32_t packed = 0xffffffffu;
            int lo = 0, hi = num_sets;                  // last set whose row starts at or before j
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_row[mid] <= j) lo = mid; else hi = mid;
            }
            const int32_t t = a.tgt_idx[j];
            if (!(s_row[lo] <= j && j < s_row[lo + 1])) {
                // (an entry that belongs to no set)
            } else if (t < t_lo || t >= t_end) {
                err |= t < 0 || t >= g.num_tensors ? kErrIdRange : kErrCrossGraph;
            } else if (from_m) {
                (void)atomicOr(&all_M[t], (u64)1 << lo);
            } else if (t < t_first) {
                lds_or(low_of(t), (u64)1 << lo);
            } else {
                lowest = min(lowest, t - t_lo);
                packed = ((uint32_t)(t - t_lo) << 6) | (uint32_t)lo;
            }
            if (!from_m) seeds[j - j0] = packed;
        }
    }
    if (boundary && tid < a.reach && t_hi - a.reach + tid >= t_first) {           // bit i: the i-th tensor of the boundary above
        lowest = t_hi - a.reach + tid - t_lo;
        seeds[tid] = ((uint32_t)lowest << 6) | (uint32_t)tid;
    } else if (boundary && tid < a.reach) {
        seeds[tid] = 0xffffffffu;
    }
    if (err) atomicOr(&s_err, err);
    lowest = -wave_max(-lowest);
    if (kSeg && lane == 0) atomicMin(&s_lowest, lowest);
    auto lowest_of = [&](int low) { return from_m ? -1 : low == 0x7fffffff ? low : t_lo + low; };        // (none: beyond every tensor)
    int32_t lowest_seed = lowest_of(lowest);
    int n_seeds = from_m || j1 < j0 ? 0 : (int)(j1 - j0);
    if (from_m) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if constexpr (kSeg) {
        if (tid >= N) return;                                // (what follows is one wave's)
        lowest_seed = lowest_of(s_lowest);
        n_seeds = boundary ? a.reach : s_own;
    }
    auto sync = [&]() {
        if constexpr (kSeg) wave_fence(); else __syncthreads();
    };
    if (from_m && seg == 0)
        for (int32_t t = t_lo + tid; t < t_first; t += N) lds_write(low_of(t), load_coherent(&all_M[t]));
    // target bits of the tensors [from, to), which the ring has come to cover.  A thread looks at the targets that it put
    // into LDS itself only if they are its wave's (the lowest one is known per wave).
    auto cover = [&](int32_t from, int32_t to) {
        if (to <= lowest_seed) return;                       // wave-uniform
        if (from_m) {
            for (int32_t t = max(from, t_mine) + tid; t < to; t += N) {
                const u64 m = load_coherent(&all_M[t]);
                if (m) lds_or(slot_of(t), m);
            }
        } else {
            for (int i = tid; i < n_seeds; i += N) {
                const uint32_t v = seeds[i];
                const int32_t t = t_lo + (int32_t)(v >> 6);
                if (v != 0xffffffffu && t >= from && t < to) lds_or(slot_of(t), (u64)1 << (v & 63));
            }
        }
    };
    cover(t_hi - R, t_hi);
    int32_t cov_lo = t_hi - R, cov_hi = cov_lo;              // tensors [cov_lo, cov_hi): their target bits are still to come
    sync();

    RingCount cnt;
#pragma unroll
    for (int p = 0; p < kRingPlanes; ++p) cnt.plane[p] = 0;
    cnt.x0 = cnt.x1 = cnt.x2 = 0;
    const int planes_used = 33 - __builtin_clz((unsigned)steps | 1u);
    const int64_t at_word = (g_lo >> 6) + gi + wd * ring_bit_words(g.num_ops, 1) + (kSeg ? seg * a.seg_words : 0);
    u64 *bits = (kSeg ? a.own_bits : a.bits) + at_word;      // this graph's words
    int32_t *cum = a.cum + at_word;
    int done = 0;                                            // operators kept in the groups so far
    int relax = 0;                                           // settling steps (statistics)
    int round = 0;
    int32_t z_hi = t_hi;                                     // the group's outputs are [z_lo, z_hi)
    if (!(W > 1 || kSeg)) first_bounds();
    if (steps > 0) ring_targets(g, cur);
    for (int step = 0; step < steps; ++step, word -= W) {
        const RingRow r = cur;
        const int32_t z_lo = __builtin_amdgcn_readfirstlane(W > 1 ? z_next : r.ob) + shift;
        const int i = word * kWave + lane;                   // this lane's operator
        const bool valid = i < n && (W == 1 || word >= 0);
        const int n_out = valid ? r.oe - r.ob : 0, n_in = valid ? r.ie - r.ib : 0;
        // fetch ahead: inputs of the next group (its bounds are here), bounds of the one after
        ring_targets(g, nxt);
        ring_bounds(in_row, out_row, nxt2, i - 2 * N, n);
        if (W > 1) z_next = at_byte(out_row, group_first(step + 1) * 4u + vz);
        u64 before = ~(u64)0;
        if (skips) before = at_byte(bits, (uint32_t)max(word, 0) * 8u + vz);

        const int32_t z0 = r.ob + shift;
        const uint32_t s0 = n_out > 0 ? slot_of(z0) : zero_at, s1 = n_out > 1 ? slot_of(z0 + 1) : zero_at;
        const int32_t wave_lo = W > 1 ? __builtin_amdgcn_readfirstlane(z0) : z_lo;       // outputs of this wave start here
        const bool many = ballot64(n_out > 2 || n_in > 4) != 0;          // some operator needs the loops over more than that
        const bool any2 = ballot64(n_in > 2) != 0, any3 = ballot64(n_in > 3) != 0;
        // Where the inputs' bits go: to the ones that the group itself writes while it settles (in), to all others when
        // it is final (out); a lane without such an input writes to a word of its own that nobody reads.
        // own: some input is written by this wave, crosses: by another wave of the group.
        bool own = false, crosses = false;
        uint32_t in[4], out[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t t = r.t[j];
            const bool is = j < n_in, inside = is && t >= z_lo;
            const uint32_t at = t >= t_first ? slot_of(t) : low_of(t);
            in[j] = inside ? at : nowhere;
            out[j] = is && !inside ? at : nowhere;
            own |= inside && t >= wave_lo;
            if (W > 1) crosses |= inside && t < wave_lo;
        }
        auto push = [&](const uint32_t (&at)[4], u64 bits) {
            lds_or(at[0], bits);
            lds_or(at[1], bits);
            if (any2) lds_or(at[2], bits);
            if (any3) lds_or(at[3], bits);
        };
        u64 k = 0, m0, m1;
        for (;;) {
            bool crossed = false;
            if (!many) {
                for (;;) {
                    m0 = lds_read(s0);
                    m1 = lds_read(s1);
                    const u64 m = m0 | m1, nb = m & ~k;
                    k = m;                                   // (the words only ever gain bits)
                    ++relax;
                    if (nb) push(in, nb);
                    if (W > 1) crossed |= nb && crosses;
                    __builtin_amdgcn_wave_barrier();
                    if (ballot64(nb && own) == 0) break;
                }
            } else {
                for (;;) {
                    m0 = lds_read(s0);
                    m1 = lds_read(s1);
                    u64 m = m0 | m1;
                    for (int j = 2; j < n_out; ++j) m |= lds_read(slot_of(z0 + j));
                    const u64 nb = m & ~k;
                    k = m;
                    ++relax;
                    bool again = nb && own;
                    if (nb) {
                        push(in, nb);
                        if (W > 1) crossed |= crosses;
                        for (int j = 4; j < n_in; ++j) {
                            const int32_t t = g.in_idx[r.ib + j];
                            if (t >= z_lo) {
                                lds_or(slot_of(t), nb);
                                again |= t >= wave_lo;
                                if (W > 1) crossed |= t < wave_lo;
                            }
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                    if (ballot64(again) == 0) break;
                }
            }
            if (W == 1) break;
            const int fl = round % 3;
            if (tid == 0) s_flag[(round + 1) % 3] = 0;
            if (ballot64(crossed) != 0 && lane == 0) s_flag[fl] = 1;
            sync();
            ++round;
            if (s_flag[fl] == 0) break;                      // the same in every thread
        }
        if (k) {                                             // the group is final
            push(out, k);
            if (many)
                for (int j = 4; j < n_in; ++j) {
                    const int32_t t = g.in_idx[r.ib + j];
                    if (t < z_lo) lds_or(t >= t_first ? slot_of(t) : low_of(t), k);
                }
        }
        cover(cov_lo, cov_hi);
        const u64 bit_word = ballot64(k != 0);
        if ((bit_word | before) != 0) {
            const uint32_t mo = (uint32_t)(z0 - t_lo) * 8u;
            if (valid) {
                at_byte(K, (uint32_t)i * 8u) = k;
                if (flags) at_byte(flags, (uint32_t)i) = k != 0;
            }
            if (n_out > 0) at_byte(M, mo) = m0;
            if (n_out > 1) at_byte(M, mo + 8) = m1;
            if (many)
                for (int j = 2; j < n_out; ++j) at_byte(M, mo + 8u * j) = lds_read(slot_of(z0 + j));
        }
        if (!kSeg && valid && a.flags2) a.flags2[o_lo + i] = k != 0;
        // the outputs' slots now stand for the tensors R below
        if (n_out > 0) lds_write(s0, 0);
        if (n_out > 1) lds_write(s1, 0);
        if (many)
            for (int j = 2; j < n_out; ++j) lds_write(slot_of(z0 + j), 0);
        cov_hi = z_hi - R;
        cov_lo = z_lo - R;
        z_hi = z_lo;
        if (!kSeg && a.pq) {
            switch (step & 3) {                              // uniform
            case 0: cnt.x0 = k; break;
            case 1: cnt.x1 = k; break;
            case 2: cnt.x2 = k; break;
            default: ring_fold(cnt, k, planes_used); break;
            }
        }
        cur = nxt;
        nxt = nxt2;
        // running count over the graph's words, highest first
        const int c = __popcll(bit_word);
        int upto = c, all = c;
        if (kSeg) {
            sync();
            if (lane == 0 && word >= 0 && !boundary) at_byte(bits, (uint32_t)word * 8u) = bit_word;
            continue;
        }
        if (W > 1) {
            if (lane == 0) s_total[wave] = c;
            sync();
            upto = all = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int cw = s_total[w];
                if (w <= wave) upto += cw;
                all += cw;
            }
        }
        if (lane == 0 && (W == 1 || word >= 0)) {
            at_byte(bits, (uint32_t)word * 8u) = bit_word;
            if (W > 1 && a.list_here) s_cum[word] = done + upto;            // operators kept in this word and above
            else at_byte(cum, (uint32_t)word * 4u) = done + upto;
        }
        done += all;
        __builtin_amdgcn_wave_barrier();
    }
    sync();
    if (kSeg) {
        // what k_ring_join needs: the bits that the segment below receives, the graph's inputs (a segment's part of them; the
        // lowest one's goes to M, where the others' are added), and the settling steps
        u64 *edge = a.edge + (((int64_t)gi * a.segs + seg) * (a.words + 1) + wd) * ring_edge_words(a);
        for (int j = tid; j < kWave; j += N) {
            const int32_t t = t_mine - a.reach + j;
            edge[j] = j < a.reach && t >= t_first ? lds_read(slot_of(t)) : 0;
        }
        if (seg == 0 && !boundary)
            for (int32_t t = t_lo + tid; t < t_first; t += N) all_M[t] = lds_read(low_of(t));
        else
            for (int32_t t = t_lo + tid; t < t_first; t += N) edge[kWave + t - t_lo] = lds_read(low_of(t));
        if (tid == 0) edge[kWave + a.low_words] = (u64)relax;
        if (seg == 0 && !boundary) {
            if (a.pq && tid < kWave) a.pq[(int64_t)(batched ? gi : wd) * 64 + tid] = 0;
            if (tid == 0) a.graphs[batched ? gi : wd] = make_int4(0, s_err, 0, found ? 1 : 0);
        }
        return;
    }
    for (int32_t t = t_lo + tid; t < t_first; t += N) all_M[t] = lds_read(low_of(t));
    if (a.pq) {
        if (steps & 3) {                                     // masks still waiting: fold them with zeros for the rest
            if ((steps & 3) < 3) cnt.x2 = 0;
            if ((steps & 3) < 2) cnt.x1 = 0;
            ring_fold(cnt, 0, planes_used);
        }
        u64 total = 0;                                       // lane q: operators of this wave's words kept for set q
#pragma unroll
        for (int p = 0; p < kRingPlanes; ++p)
            if (p < planes_used)                             // wave-uniform
                total += (u64)__popcll(wave_transpose64(cnt.plane[p])) << p;
        if (W > 1) {                                         // (the ring is free now; it has at least N words)
            ring[tid] = total;
            sync();
            total = 0;
            if (wave == 0)
                for (int w = 0; w < W; ++w) total += ring[w * kWave + lane];
        }
        if (wave == 0) a.pq[(int64_t)blockIdx.x * 64 + lane] = (int64_t)total;
    }
    if (lane == 0) atomicAdd(&s_relax, relax);
    sync();
    if (tid == 0) {
        const int4 st = make_int4(done, s_err, s_relax, found ? 1 : 0);
        a.graphs[blockIdx.x] = st;
        if (!batched) a.kept_count[wd] = done;
        if (W > 1 && a.list_here) ring_finish(a, st);
    }
    if (W > 1 && a.list_here) {
        // A small single graph: the ordered list right here, one launch and one gap less (2 000 operators: 52 -> 49 us).
        // Every wave takes the words that it swept, four in flight, and reads back what its own lanes stored.
        int w = n_words - 1 - wave;
        for (int step = 0; step < steps; step += 4, w -= 4 * W) {
            u64 k[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = (w - c * W) * kWave + lane;
                k[c] = step + c < steps && w - c * W >= 0 && i < n ? K[i] : 0;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const u64 kept = ballot64(k[c] != 0);
                if (kept == 0) continue;                     // (also past the last word)
                const int pos = done - s_cum[w - c * W] + __popcll(kept & lanemask_lt());
                if (k[c]) {
                    a.kept_ops[pos] = (w - c * W) * kWave + lane;
                    if (a.kept_masks) a.kept_masks[pos] = k[c];
                }
            }
        }
    }
}

// Packed batch: kept_count[1 + g] = operators kept in the graphs before g, [1 + G] and [0] = in all; error bits of all
// graphs and the largest number of settling steps go to the entry behind the last graph's.  One workgroup.
__global__ __launch_bounds__(1024) void k_ring_offsets(RingArgs a)
{
    __shared__ int wtot[16], s_err, s_relax;
    const int lane = lane_id(), wave = threadIdx.x >> 6, G = a.g.num_graphs;
    if (threadIdx.x == 0) s_err = s_relax = 0;
    __syncthreads();
    const int per = (G + 1023) / 1024, lo = min((int)threadIdx.x * per, G), hi = min(lo + per, G);
    int sum = 0, err = 0, relax = 0;
    for (int i = lo; i < hi; ++i) {
        const int4 v = a.graphs[i];
        sum += v.x;
        err |= v.y;
        relax = max(relax, v.z);
    }
    if (err) atomicOr(&s_err, err);
    const int wrelax = wave_max(relax);
    if (lane == 0) atomicMax(&s_relax, wrelax);
    const int incl = wave_incl_scan(sum);
    if (lane == kWave - 1) wtot[wave] = incl;
    __syncthreads();
    int run = incl - sum, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < wave) run += wtot[w];
        all += wtot[w];
    }
    for (int i = lo; i < hi; ++i) {
        a.kept_count[1 + i] = run;
        run += a.graphs[i].x;
    }
    if (threadIdx.x == 0) {
        a.kept_count[1 + G] = all;
        a.kept_count[0] = all;
        a.graphs[G] = make_int4(all, s_err, s_relax, a.graphs[0].w);
    }
}

// Ordered compaction from the words and running counts of the sweep: the position of a kept operator is known from its
// word alone, so a wave takes any four words of its graph at a time.  Memory bounds it: neighbouring words go to one wave and
// neighbouring waves, so that the lines that two words share are written at one time in one cache (4 096 graphs of 20 000 operators:
// 345 us with the words dealt to the waves in turn, 298 = 4.5 TB/s so).  The first workgroup also leaves the header for recycling and
// hands the status to the host.
constexpr int kRingScatterThreads = 256;

__global__ __launch_bounds__(kRingScatterThreads) void k_ring_scatter(RingArgs a)
{
    const GraphView &g = a.g;
    const int lane = lane_id();
    const bool batched = g.num_graphs > 1;
    const int gi = batched ? blockIdx.x : 0, wd = batched ? 0 : blockIdx.x;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        int4 st = a.graphs[batched ? g.num_graphs : 0];
        for (unsigned w = 1; !batched && w < gridDim.x; ++w) {       // words of sets: errors of all, settling steps added up
            const int4 more = a.graphs[w];
            st.y |= more.y;
            st.z += more.z;
        }
        ring_finish(a, st);
    }
    const int64_t o_lo = batched ? g.op_off[gi] : 0, o_hi = batched ? g.op_off[gi + 1] : g.num_ops;
    if (o_hi <= o_lo) return;
    const int64_t first = (o_lo >> 6) + gi + wd * ring_bit_words(g.num_ops, 1);              // the graph's words
    const int64_t n_words = (o_hi - o_lo + kWave - 1) >> 6;
    const int64_t end = a.kept_count[batched ? gi + 2 : wd];
    const u64 *K = a.K + (int64_t)wd * g.num_ops;
    int32_t *kept_ops = a.kept_ops + (int64_t)wd * g.num_ops;
    u64 *kept_masks = a.kept_masks ? a.kept_masks + (int64_t)wd * g.num_ops : nullptr;
    constexpr int kStep = kRingScatterThreads / kWave * 4;
    const int64_t per = ((n_words + gridDim.y - 1) / gridDim.y + kStep - 1) / kStep * kStep;  // words of this workgroup
    const int64_t stop = min(n_words, (blockIdx.y + 1) * per);
    for (int64_t w0 = blockIdx.y * per + (threadIdx.x >> 6) * 4; w0 < stop; w0 += kStep) {
        u64 bits[4], k[4];
        int cum[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t w = w0 + c;
            bits[c] = w < stop ? a.bits[first + w] : 0;
            cum[c] = w < stop ? a.cum[first + w] : 0;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool has = (bits[c] >> lane) & 1;
            k[c] = has && kept_masks ? K[o_lo + (w0 + c) * kWave + lane] : 0;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if ((bits[c] >> lane) & 1) {
                const int64_t pos = end - cum[c] + __popcll(bits[c] & lanemask_lt());
                kept_ops[pos] = (int32_t)(o_lo + (w0 + c) * kWave + lane);
                if (kept_masks) kept_masks[pos] = k[c];
            }
        }
    }
}

// ---- segments ---------------------------------------------------------------------------------------------------------
// "The OR of those of 64 words that a mask names", the words in the lanes of a wave, alone or in pairs: table n gives the OR of
// any of the words 4n .. 4n + 3, so that a mask takes sixteen look-ups.  The sixteen entries of a table lie in 64 different banks,
// and lanes that want the same one share the read; entry v of table n sits at v ^ (n mod 4), which spreads the writes as well.
struct alignas(16) RingPair { u64 m, through; };
constexpr int kPairTable = 16 * 16;

__device__ __forceinline__ u64 word_or(u64 a, u64 b) { return a | b; }
__device__ __forceinline__ RingPair word_or(const RingPair &a, const RingPair &b) { return {a.m | b.m, a.through | b.through}; }
// word k of the four lanes that this one is among
template <int k> __device__ __forceinline__ u64 word_of_four(u64 v)
{
    const uint32_t lo = (uint32_t)dpp_move<k * 0x55, 0xf>(0, (int)(uint32_t)v), hi = (uint32_t)dpp_move<k * 0x55, 0xf>(0, (int)(uint32_t)(v >> 32));
    return ((u64)hi << 32) | lo;
}
template <int k> __device__ __forceinline__ RingPair word_of_four(const RingPair &v) { return {word_of_four<k>(v.m), word_of_four<k>(v.through)}; }

template <typename Word> __device__ __forceinline__ void ring_table(Word *table, const Word &word)
{
    const int lane = lane_id(), place = (lane >> 2) & 3;
    const Word p0 = word_of_four<0>(word), p1 = word_of_four<1>(word), p2 = word_of_four<2>(word), p3 = word_of_four<3>(word);
    const Word high = word_or(lane & 1 ? p2 : Word{}, lane & 2 ? p3 : Word{});
    Word *to = table + lane * 4;                             // entries 4 (l mod 4) .. + 3 of table l / 4
    to[place] = high;
    to[place ^ 1] = word_or(high, p0);
    to[place ^ 2] = word_or(high, p1);
    to[place ^ 3] = word_or(word_or(high, p0), p1);
    wave_fence();
}

template <typename Word> __device__ __forceinline__ Word ring_named(const Word *table, u64 mask)
{
    Word r{};
    mask ^= 0x3210321032103210ull;                           // (n mod 4 in every nibble)
#pragma unroll
    for (int n = 0; n < 16; ++n) r = word_or(r, table[n * 16 + (int)((mask >> (4 * n)) & 15)]);
    return r;
}

// M of the boundaries between a graph's segments.  What segment q sends below is own(q) | the words of the boundary above it
// that through(q) names: an affine map of 64 words, and the map of several segments in a row is of the same kind.  Each of
// eight waves folds the segments of an eighth of the graph into one map, the first wave goes through the eight, and then
// every wave once more through its own with what comes in from above.  LDS bounds the folding (a step of all eight: 1 600
// cycles of it), its latency the rest (some 500 cycles a step).  79 segments: one wave from the top to the bottom 40 us, sixteen
// that fold and combine in four rounds 15.
//   at(q, word) -> lane's entry of a segment's edge (the second word: through); take(q, m) is given M of the boundary above q.
constexpr int kCarryThreads = 1024, kCarryWaves = 8;
struct CarryLds {
    RingPair table[kCarryWaves][kPairTable];
    RingPair row[kCarryWaves][kWave];
    u64 above[kCarryWaves][kWave];
};

template <typename At, typename Take>
__device__ __forceinline__ void ring_carry(int segs, CarryLds &lds, At at, Take take)
{
    constexpr int kHeld = 4;                                 // segments ahead (a load takes as long as two or three steps)
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per = (segs + kCarryWaves - 1) / kCarryWaves, parts = (segs + per - 1) / per;
    const int top = segs - 1 - wave * per, mine = wave < parts ? min(per, top + 1) : 0;      // this wave's: top, top - 1, ...
    RingPair *table = lds.table[wave & (kCarryWaves - 1)];
    u64 *table1 = reinterpret_cast<u64 *>(table);
    RingPair held[kHeld];
    auto fetch = [&](int j) -> RingPair {
        const int q = max(top - j, 0);
        return {at(q, false), q + 1 < segs ? at(q, true) : 0};                       // (nothing comes in at the top)
    };
    auto fetch_first = [&]() {
#pragma unroll
        for (int j = 0; j < kHeld; ++j) held[j] = fetch(j);
    };
    auto next = [&](int j) -> RingPair {                     // the j-th, and another one on its way
        const RingPair r = held[0];
#pragma unroll
        for (int i = 0; i + 1 < kHeld; ++i) held[i] = held[i + 1];
        held[kHeld - 1] = fetch(j + kHeld);
        return r;
    };
    RingPair all{};                                          // the map of this wave's segments so far
    if (mine > 0) {
        fetch_first();
        all = next(0);
#pragma unroll 1
        for (int j = 1; j < mine; ++j) {
            const RingPair seg = next(j);
            ring_table(table, all);
            all = ring_named(table, seg.through);
            all.m |= seg.m;
        }
        lds.row[wave][lane] = all;
        fetch_first();
    }
    __syncthreads();
    if (wave == 0) {
        u64 m = all.m;
#pragma unroll 1
        for (int v = 1; v < parts; ++v) {
            lds.above[v][lane] = m;
            const RingPair part = lds.row[v][lane];
            ring_table(table1, m);
            m = part.m | ring_named(table1, part.through);
        }
        lds.above[0][lane] = 0;
    }
    __syncthreads();
    if (mine == 0) return;
    u64 m = lds.above[wave][lane];
#pragma unroll 1
    for (int j = 0;; ++j) {
        take(top - j, m);
        if (j + 1 == mine) break;
        const RingPair seg = next(j);
        ring_table(table1, m);
        m = seg.m | ring_named(table1, seg.through);
    }
}

// Batches: M of the boundary above every segment of a graph, and the operators that its segments keep.  A workgroup per
// graph.
__global__ __launch_bounds__(kCarryThreads) void k_ring_carry(RingArgs a)
{
    __shared__ CarryLds s_carry;
    __shared__ u64 s_reached[kRingMaxSegs];
    __shared__ int s_kept[kRingMaxSegs], s_all;
    const GraphView &g = a.g;
    const int gi = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t o_lo = g.op_off[gi];
    const int n = (int)(g.op_off[gi + 1] - o_lo), n_words = (n + kWave - 1) >> 6;
    const int segs = (n_words + a.seg_words - 1) >> a.seg_shift;
    for (int q = tid; q < segs; q += kCarryThreads) s_kept[q] = 0;
    if (tid == 0) s_all = 0;
    const int64_t step = ring_edge_words(a);
    u64 *edge = a.edge + (int64_t)gi * a.segs * 2 * step + lane;
    if (segs > 0)
        ring_carry(segs, s_carry, [&](int q, bool through) { return edge[(q * 2 + through) * step]; },
                   [&](int q, u64 m) {
                       edge[q * 2 * step] = m;              // (in the place of what it sends below, which has been fetched)
                       const u64 reached = ballot64(m != 0);
                       if (lane == 0) s_reached[q] = reached;
                   });
    __syncthreads();
    const u64 *own = a.own_bits + (o_lo >> 6) + gi;
    for (int w0 = wave; w0 < n_words; w0 += 4 * (kCarryThreads / kWave)) {
        u64 bits[4], b[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int w = w0 + c * (kCarryThreads / kWave), i = w * kWave + lane;
            const u64 reached = w < n_words ? s_reached[w >> a.seg_shift] : 0;
            bits[c] = w < n_words ? own[w] : 0;
            b[c] = reached && i < n ? a.b_K[o_lo + i] & reached : 0;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int w = w0 + c * (kCarryThreads / kWave);
            const int kept = __popcll(bits[c] | ballot64(b[c] != 0));
            if (lane == 0 && kept) atomicAdd(&s_kept[w >> a.seg_shift], kept);
        }
    }
    __syncthreads();
    int kept = 0;
    for (int q = tid; q < segs; q += kCarryThreads) {
        a.seg_kept[(int64_t)gi * a.segs + q] = s_kept[q];
        kept += s_kept[q];
    }
    kept = wave_sum(kept);
    if (lane == 0 && kept) atomicAdd(&s_all, kept);
    __syncthreads();
    if (tid == 0) a.graphs[gi].x = s_all;
}

// The result of a segment: what its own targets gave (k_ring_sweep) and what its boundary brings in; and its part of the
// ordered list.  A single graph's workgroups each work out the boundaries, and the operators kept before theirs, on their
// own, which takes less time than another launch.
constexpr int kJoinThreads = 512;

template <bool kBatch>
__global__ __launch_bounds__(kBatch ? kJoinThreads : kCarryThreads) void k_ring_join(RingArgs a)
{
    constexpr int N = kBatch ? kJoinThreads : kCarryThreads, W = N / kWave;
    constexpr int kBelow = kBatch ? 1 : 8;                   // words before the segment that a wave has in flight
    __shared__ u64 s_reached[kBatch ? 1 : kRingMaxSegs], s_table[kPairTable], s_own;
    __shared__ int s_part[W], s_err[W], s_relax[W], s_count[kRingMaxSegWords], s_sets[kWave];
    const GraphView &g = a.g;
    const int gi = blockIdx.x, seg = blockIdx.y, wd = blockIdx.z, tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t g_lo = kBatch ? g.op_off[gi] : 0;
    const int n_all = (int)((kBatch ? g.op_off[gi + 1] : g.num_ops) - g_lo);
    const int all_words = (n_all + kWave - 1) >> 6, segs = (all_words + a.seg_words - 1) >> a.seg_shift;
    if (seg > 0 && seg >= segs) return;
    const int first_word = seg * a.seg_words, first = first_word * kWave;
    const int n = min(n_all - first, a.seg_words * kWave), n_words = (n + kWave - 1) >> 6;
    const int64_t o_lo = g_lo + first;
    const int64_t step = ring_edge_words(a), per_word = ring_bit_words(g.num_ops, 1);
    const u64 *edge = a.edge + (int64_t)gi * a.segs * (a.words + 1) * step;
    const u64 *own_bits = a.own_bits + (g_lo >> 6) + gi + wd * per_word;
    const int32_t t_lo = kBatch ? (int32_t)g.t_off[gi] : 0, t_end = kBatch ? (int32_t)g.t_off[gi + 1] : g.num_tensors;
    const int32_t shift = t_end - g.out_rowptr[g_lo + n_all], t_first = g.out_rowptr[g_lo] + shift;
    const int32_t t_mine = g.out_rowptr[o_lo] + shift, t_hi = g.out_rowptr[o_lo + n] + shift;
    u64 *K = a.K + (int64_t)wd * g.num_ops + o_lo, *M = a.M + (int64_t)wd * g.num_tensors;
    const u64 *b_K = a.b_K + o_lo;
    const bool top = seg + 1 >= segs;                        // (nothing comes in, and nothing was written to b_K and b_M)
    if (tid < kWave) s_sets[tid] = 0;
    // a wave's first word of operators and run of tensors are on their way meanwhile
    const int i0 = wave * kWave + lane;
    const int32_t t0 = t_mine + wave * kWave + lane;
    const u64 K0 = i0 < n ? K[i0] : 0, b_K0 = !top && i0 < n ? b_K[i0] : 0;
    const u64 M0 = t0 < t_hi ? M[t0] : 0, b_M0 = !top && t0 < t_hi ? a.b_M[t0] : 0;

    // M of the boundary above this segment, and how many operators are kept before it
    int before = 0;
    if constexpr (kBatch) {
        if (wave == 0) {
            const u64 m = segs > 0 ? edge[seg * 2 * step + lane] : 0;
            const u64 reached = ballot64(m != 0);
            if (lane == 0) s_own = reached;
            ring_table(s_table, m);
        }
        for (int i = tid; i < gi; i += N) before += a.graphs[i].x;
        for (int q = tid; q < seg; q += N) before += a.seg_kept[(int64_t)gi * a.segs + q];
    } else {
        __shared__ CarryLds s_carry;
        u64 bits, b[kBelow];                                 // (lane c: of the c-th word)
        auto fetch = [&](int w0) {
            bits = lane < kBelow && w0 + lane * W < first_word ? own_bits[w0 + lane * W] : 0;
#pragma unroll
            for (int c = 0; c < kBelow; ++c) b[c] = w0 + c * W < first_word ? a.b_K[(w0 + c * W) * kWave + lane] : 0;
        };
        fetch(wave);
        const u64 *e = edge + lane;
        const int64_t through_at = (int64_t)(a.words - wd) * step;
        ring_carry(segs, s_carry,
                   [&](int q, bool through) { return e[((int64_t)q * (a.words + 1) + wd) * step + (through ? through_at : 0)]; },
                   [&](int q, u64 m) {
                       const u64 reached = ballot64(m != 0);
                       if (lane == 0) s_reached[q] = reached;
                       if (q != seg) return;
                       if (lane == 0) s_own = reached;
                       ring_table(s_table, m);
                   });
        __syncthreads();
        for (int w0 = wave; w0 < first_word; w0 += kBelow * W) {
            if (w0 != wave) fetch(w0);
#pragma unroll
            for (int c = 0; c < kBelow; ++c) {
                const int w = w0 + c * W;
                const u64 reached = w < first_word ? s_reached[w >> a.seg_shift] : 0;
                const u64 kept = ballot64((b[c] & reached) != 0);
                before += lane == c ? __popcll(bits | kept) : 0;
            }
        }
    }
    before = wave_sum(before);
    if (lane == 0) s_part[wave] = before;
    __syncthreads();
    const u64 reached = s_own;                               // tensors of the boundary that carry anything
    before = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) before += s_part[w];

    // operators kept per word of this segment
    for (int w = wave; w < n_words; w += W) {
        const int i = w * kWave + lane;
        const u64 b = w == wave ? b_K0 & reached : reached && i < n ? b_K[i] & reached : 0;
        const u64 kept = own_bits[first_word + w] | ballot64(b != 0);
        if (lane == 0) {
            a.bits[(g_lo >> 6) + gi + wd * per_word + first_word + w] = kept;
            s_count[w] = __popcll(kept);
        }
    }
    __syncthreads();
    int all = 0;
    if (wave == 0) {                                         // running count over the words
        for (int w = 0; w < n_words; w += kWave) {
            const int c = w + lane < n_words ? s_count[w + lane] : 0;
            const int upto = wave_incl_scan(c);
            if (w + lane < n_words) s_count[w + lane] = all + upto - c;
            all += __builtin_amdgcn_readlane(upto, kWave - 1);
        }
    }
    __syncthreads();

    // operators: masks, flags, list
    uint8_t *flags = a.flags ? a.flags + (int64_t)wd * g.num_ops + o_lo : nullptr;
    uint8_t *flags2 = a.flags2 ? a.flags2 + (int64_t)wd * g.num_ops + o_lo : nullptr;
    int32_t *kept_ops = a.kept_ops + (int64_t)wd * g.num_ops;
    u64 *kept_masks = a.kept_masks ? a.kept_masks + (int64_t)wd * g.num_ops : nullptr;
    int sets = 0;                                            // lane q: operators of this wave kept for set q
    for (int w = wave; w < n_words; w += W) {
        const int i = w * kWave + lane;
        u64 k = w == wave ? K0 : i < n ? K[i] : 0;
        if (reached) {
            const u64 b = w == wave ? b_K0 & reached : i < n ? b_K[i] & reached : 0;
            if (ballot64(b != 0) != 0) {
                const u64 more = ring_named(s_table, b);
                if (more & ~k) K[i] = k | more;
                k |= more;
            }
        }
        if (i < n && flags) flags[i] = k != 0;
        if (i < n && flags2) flags2[i] = k != 0;
        const u64 kept = ballot64(k != 0);
        if (kept == 0) continue;
        if (k) {
            const int64_t pos = (int64_t)before + s_count[w] + __popcll(kept & lanemask_lt());
            kept_ops[pos] = (int32_t)(o_lo + i);
            if (kept_masks) kept_masks[pos] = k;
        }
        if (a.pq) sets += __popcll(wave_transpose64(k));
    }
    if (a.pq && sets) atomicAdd(&s_sets[lane], sets);
    // tensors
    if (reached) {
        for (int32_t first_t = t_mine + wave * kWave; first_t < t_hi; first_t += N) {
            const int32_t t = first_t + lane;
            const bool held = first_t - t_mine < N;
            const u64 b = held ? b_M0 & reached : t < t_hi ? a.b_M[t] & reached : 0, has = held ? M0 : t < t_hi ? M[t] : 0;
            if (ballot64(b != 0) == 0) continue;
            const u64 more = ring_named(s_table, b);
            if (more & ~has) M[t] = has | more;
        }
    }
    // the graph's inputs: every segment's part goes to where the lowest one has put its own
    const u64 *own = edge + ((int64_t)seg * (a.words + 1) + wd) * step + kWave, *through = own + (int64_t)(a.words - wd) * step;
    for (int32_t i = tid; i < t_first - t_lo; i += N) {
        u64 v = seg > 0 ? own[i] : 0;
        if (reached) v |= ring_named(s_table, through[i] & reached);
        if (v) (void)atomicOr(&M[t_lo + i], v);
    }
    __syncthreads();
    if (a.pq && tid < kWave && s_sets[tid])
        (void)atomicAdd(reinterpret_cast<u64 *>(&a.pq[(int64_t)(kBatch ? gi : wd) * 64 + tid]), (u64)s_sets[tid]);
    if (kBatch) {
        if (tid == 0 && seg == 0) a.kept_count[1 + gi] = before;
        if (gi != g.num_graphs - 1 || !top) return;
        if (tid == 0) a.kept_count[0] = a.kept_count[1 + g.num_graphs] = (int64_t)before + all;
    } else {
        if (!top) return;
        if (tid == 0) a.kept_count[wd] = (int64_t)before + all;
        if (wd > 0) return;
    }
    // the last workgroup of the first word: what went wrong, settling steps where somebody asks, and the header for recycling
    int err = 0, relax = 0;
    const int rows = kBatch ? g.num_graphs : a.words;
    for (int i = tid; i < rows; i += N) err |= a.graphs[i].y;
    if (a.count_steps) {
        const int per_seg = a.words + 1;
        for (int j = 0; j < g.num_graphs; ++j) {
            const int ops = (int)(kBatch ? g.op_off[j + 1] - g.op_off[j] : g.num_ops);
            const int sweeps = ((((ops + kWave - 1) >> 6) + a.seg_words - 1) >> a.seg_shift) * per_seg - 1;  // (none above the last)
            for (int i = tid; i < sweeps; i += N)
                relax += (int)a.edge[((int64_t)j * a.segs * per_seg + i) * step + kWave + a.low_words];
        }
    }
    err = __builtin_amdgcn_readlane(wave_incl_or(err), kWave - 1);
    relax = wave_sum(relax);
    if (lane == 0) {
        s_err[wave] = err;
        s_relax[wave] = relax;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < W; ++w) {
            err |= s_err[w];
            relax += s_relax[w];
        }
        ring_finish(a, make_int4(0, err, relax, a.graphs[0].w));
    }
}

size_t ring_segment_scratch(RingArgs &a, void *mem)
{
    char *p = static_cast<char *>(mem);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += (bytes + 255) & ~(size_t)255;
        return r;
    };
    const GraphView &g = a.g;
    const size_t G = (size_t)g.num_graphs, words = (size_t)a.words, segs = (size_t)a.segs;
    a.b_M = reinterpret_cast<u64 *>(take((size_t)g.num_tensors * 8));
    a.b_K = reinterpret_cast<u64 *>(take((size_t)g.num_ops * 8));
    a.edge = reinterpret_cast<u64 *>(take(G * segs * (words + 1) * (size_t)ring_edge_words(a) * 8));
    a.own_bits = reinterpret_cast<u64 *>(take((size_t)ring_bit_words(g.num_ops, (int64_t)G) * words * 8));
    a.seg_kept = reinterpret_cast<int32_t *>(take(G > 1 ? G * segs * 4 : 0));
    return off;
}

template <int W, int H> static hipError_t launch_ring_w(const RingArgs &a, size_t lds, hipStream_t s)
{
    constexpr bool kSeg = H > 0;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_ring_sweep<W, H>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRingMaxLds);
        if (e != hipSuccess) return e;
    }
    const unsigned rows = (unsigned)(a.g.num_graphs > 1 ? a.g.num_graphs : a.words);
    const dim3 grid = kSeg ? dim3((unsigned)a.g.num_graphs, (unsigned)a.segs, (unsigned)a.words + 1) : dim3(rows);
    hipLaunchKernelGGL((k_ring_sweep<W, H>), grid, dim3((H > W ? H : W) * kWave), lds, s, a);
    return hipGetLastError();
}

constexpr int64_t kRingListOps = 16384;

hipError_t launch_ring_sweep(RingArgs a, int waves, int dist, int span64, int64_t max_graph_ops, int *launches, hipStream_t s,
                             hipEvent_t *ev, bool all)
{
    a.ring_words = (int32_t)ring_words(a.segs > 1 ? kRingSegWaves : waves, dist, span64);
    const int G = a.g.num_graphs;
    const int64_t words = (max_graph_ops + 63) / 64 + 1;
    size_t lds = (size_t)(a.ring_words + a.low_words + kRingExtraWords) * sizeof(u64) + (size_t)a.seed_words * sizeof(uint32_t);
    // (a wave of the sweep takes four words in 1.2 us, the launch of a pass of its own costs 6: up to about 20 words per wave)
    a.list_here = a.segs <= 1 && G == 1 && a.words == 1 && waves > 1 && max_graph_ops <= kRingListOps && lds + (size_t)words * sizeof(int) <= kRingMaxLds;
    if (a.list_here) lds += (size_t)words * sizeof(int);
    hipError_t e = a.segs > 1 ? (a.few_segs ? launch_ring_w<kRingSegWaves, kRingPlaceWaves>(a, lds, s) : launch_ring_w<kRingSegWaves, 1>(a, lds, s))
                 : waves == 1 ? launch_ring_w<1, 0>(a, lds, s) : waves == 4 ? launch_ring_w<4, 0>(a, lds, s) : launch_ring_w<16, 0>(a, lds, s);
    *launches = a.list_here ? 1 : G > 1 ? 3 : 2;
    auto mark = [&](int i) {
        if (e == hipSuccess && ev && (i == 0 || all)) e = hipEventRecord(ev[i], s);
    };
    mark(0);
    if (e != hipSuccess) return e;
    if (G > 1) {
        if (a.segs > 1) hipLaunchKernelGGL(k_ring_carry, dim3((unsigned)G), dim3(kCarryThreads), 0, s, a);
        else hipLaunchKernelGGL(k_ring_offsets, dim3(1), dim3(1024), 0, s, a);
        e = hipGetLastError();
    }
    mark(1);
    if (e != hipSuccess) return e;
    if (a.list_here) {
        mark(2);
        return e;
    }
    if (a.segs > 1) {
        const dim3 grid((unsigned)G, (unsigned)a.segs, (unsigned)a.words);
        if (G > 1) hipLaunchKernelGGL(k_ring_join<true>, grid, dim3(kJoinThreads), 0, s, a);
        else hipLaunchKernelGGL(k_ring_join<false>, grid, dim3(kCarryThreads), 0, s, a);
        e = hipGetLastError();
        mark(2);
        return e;
    }
    // a wave per 16 words of the largest graph, four in flight; per 4 words, one round trip each, while that fits the chip
    const int64_t rows = G > 1 ? G : a.words;
    const int64_t per = rows * ((words + 15) / 16) <= 2048 ? 16 : 64;
    int64_t split = (words + per - 1) / per;
    if (split > 256) split = 256;
    const dim3 grid((unsigned)rows, (unsigned)split);
    hipLaunchKernelGGL(k_ring_scatter, grid, dim3(kRingScatterThreads), 0, s, a);
    e = hipGetLastError();
    mark(2);
    return e;
}

}  // namespace dgn
