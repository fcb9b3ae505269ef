// Descending sweep of one graph whose operators come in layers: recorded in order, hundreds of neighbouring operators that do not
// read each other, and what they read not more than some tens of layers back.
//
// Level by level such a graph costs a launch and a chain of memory accesses per few layers, and its operators are processed
// several times.  Here a workgroup walks all of it, from the highest operator down, a step of up to 512 neighbouring operators
// at a time, none of which reads from the same step: every operator is processed once, after all its readers, and what the
// steps hand on -- M of the tensors around the place that has been reached -- stays in LDS.  Sixteen sets to a workgroup
// (two bytes per tensor, so that 49 152 of them fit), which sweep side by side: sets have nothing to do with each other.
//   k_band_plan cuts the operators into steps and packs what the sweep needs of an operator into 12 bytes (LDS slots of its
// outputs and inputs).  A step that ends before operator b may begin at any operator behind the last one that some operator
// before b reads from (in its segment of 8 192 operators): a running maximum, and then a chain of one LDS access per step.
// Its other workgroups clear M.
//   k_band_sweep: eight waves process a step's operators (two LDS reads, up to four ORs), the other eight take M of the
// step before out of LDS to memory, and put target bits, which they hold in registers, in place two steps ahead (a call of
// more than 2 048 targets, of all its words, sends them by way of M and the seed kernel, since one workgroup may own them all: steps of
// 0.35 us instead of 0.27).  Operators are fetched eight steps ahead; no step waits for memory, and
// a barrier is all that separates two of them.  The removal rule's passes follow and take K from M: keeping K of a step in LDS and storing
// it from here cost the sweep 19 us of 161; the count pass's two reads per operator cost 4 more (7.8 -> 11.7), the list 1.
//
// What bounds it: the instructions of a step, 0.27 us for 400 operators, one wave's after the other's: barrier and bounds
// 0.15, ORs 0.04, the flush's stores (two bytes every eight; in runs of their own as long) 0.03.  500 layers of 400 operators, 64 sets, 525 steps: plan
// 20 us, sweep 142, count and list 24, whole prune 370 -> 201; 300 of 800 412 -> 223; 200 of 90 170 -> 110; 1 000 of 800, 16 sets, 576.  On
// the way: bounds of eight steps held in a register instead of LDS reads 168 against 161; target bits read back from M a step at a time 218, looked
// for among the held ones in every step 225 (now a scalar compare), addresses by the vector unit instead of buffer offsets 219, whole prune, when it took 215.
//
// What a graph must satisfy the plan finds out on the device: outputs numbered as they are created, in one run up to the last
// tensor, inputs written before, at most kBandMaxSteps steps, of kBandMeanOps operators or more on average where there are more than
// kBandFewSteps, and everything read no further back than LDS holds.  If not, nothing but the clear has happened, and the host traverses the graph level by level instead, now and
// from then on.  Which graphs are tried: kBandSoonShare and band_most_ops in api.hip.
#include "common.h"

namespace dgn {

constexpr int kBandSegOps = 8192;                   // operators planned by a workgroup
constexpr int kBandSegSteps = 512;                  // their steps, at most
constexpr int kBandRing = 49152;                    // tensors in LDS: tensor t at slot t mod kBandRing,
constexpr int kBandNowhere = kBandRing + kBandMaxLow;                  // graph input t at kBandRing + t; slots that nobody reads
constexpr int kBandZero = kBandNowhere + 2 * kWave;                    // one that stays zero
constexpr int kBandStepsAt = (kBandZero + 4) / 2;             // (in 4-byte words) the steps' first operators and tensors
constexpr int kBandPad = 32;                        // empty ones behind them
constexpr int kBandMaxSegs = (int)(kBandMaxOps / kBandSegOps);
constexpr size_t kBandLds = ((size_t)kBandStepsAt + 2 * (kBandMaxSteps + 1 + kBandPad) + kBandMaxSegs + 8 + 18) * sizeof(uint32_t);
constexpr uint32_t kBandMore = 0xffff;
static_assert(kBandZero < kBandMore, "slots have 16 bits");
static_assert(kBandLds <= kRingMaxLds, "LDS of a compute unit");
constexpr int kBandPlanThreads = 1024, kBandPer = kBandSegOps / kBandPlanThreads;
constexpr int kBandHalf = kBandStepOps;             // threads for operators, and as many for tensors (two each)
constexpr int kBandFewSteps = 64, kBandMeanOps = 24;          // any graph in so few steps, others with so many operators to a step
constexpr int kBandHeld = 4;                        // targets of sixteen sets that a thread keeps
static_assert(kBandMaxTargets <= kBandHeld * kBandHalf, "all of a call in one workgroup");
constexpr int kBandAhead = 8;                      // steps that loads are ahead
// Slots are used again.  Those of a step's tensors are zero two barriers behind the step that follows it: from the third step on for operators,
// which reach s_dist below the end of theirs (k_band_sweep asks for s_dist and four spans), and for target bits, put in place two steps ahead, here:
static_assert(5 * kBandStepOuts <= kBandRing, "target bits go into slots that are zero");
static_assert(kBandPad >= 3 * kBandAhead + 6, "bounds are read so far behind the last step");

constexpr int kEntryBytes = 12;
typedef uint32_t Entry __attribute__((ext_vector_type(3)));
constexpr int kBufferWord = 0x00020000;             // raw buffer of 32-bit elements, stride 0
constexpr int kPastEnd = 0x7fff0000;                // beyond every buffer here

__device__ __forceinline__ uint32_t band_slot(int32_t t, int32_t t_first)
{
    return t < t_first ? (uint32_t)(kBandRing + t) : (uint32_t)t % (uint32_t)kBandRing;
}

// Entry of an operator, six slots of two bytes: its first two outputs (the first twice, if it is the only one; a slot that stays zero), its first four inputs
// (absent ones: a slot of its own that nobody reads); more outputs or inputs than that: kBandMore in the place of the last one.
// 200 000 operators, 25 workgroups: 20 us, half of it instructions of the few compute units at work, the rest latency.
__global__ __launch_bounds__(kBandPlanThreads) void k_band_plan(BandArgs a)
{
    __shared__ int32_t s_begin[kBandSegOps];        // by operator: the last one read from; then where a step that ends behind it begins
    __shared__ uint16_t s_out[kBandSegOps + 1];     // outputs of the segment's operators before
    __shared__ int32_t s_list[kBandSegSteps + 1];
    __shared__ int s_wave[kBandPlanThreads / kWave], s_bad, s_dist, s_span, s_steps;
    const GraphView &g = a.g;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int num_segs = (g.num_ops + kBandSegOps - 1) / kBandSegOps;
    if ((int)blockIdx.x >= num_segs) {              // the other workgroups clear
        const size_t at = (size_t)(blockIdx.x - num_segs) * kBandPlanThreads + tid, stride = (size_t)(gridDim.x - num_segs) * kBandPlanThreads;
        for (int r = 0; r < kBandRegions; ++r) {
            u64 *p = static_cast<u64 *>(a.clear[r].ptr);
            if (!p) continue;
            for (size_t i = at; i < a.clear[r].bytes / 8; i += stride) p[i] = 0;
        }
        return;
    }
    const int32_t lo = (int32_t)blockIdx.x * kBandSegOps, n = min(kBandSegOps, g.num_ops - lo);
    const int32_t shift = g.num_tensors - g.nnz_out;        // output edge e should be tensor e + shift; the ones below are graph inputs
    const int32_t first_out = g.out_rowptr[lo];
    if (tid == 0) s_bad = s_dist = s_span = s_steps = 0;
    if (blockIdx.x == 0 && tid == 0) {
        a.host_status[kBandFound] = a.recycle && same_header(*a.hdr, a.want);
        a.hdr->magic = 0;                                   // (the last pass of the compaction writes a new one)
    }
    __syncthreads();
    bool bad = shift < 0;
    int dist = 0;
    // every access of all of a thread's operators in flight at once (lanes past the end: the last operator's)
    int4 rec[kBandPer];
    int32_t ob[kBandPer], oe[kBandPer], newest[kBandPer];
#pragma unroll
    for (int j = 0; j < kBandPer; ++j) {
        const int32_t o = lo + min(j * kBandPlanThreads + tid, n - 1);
        rec[j] = op_record(g, o);
        ob[j] = g.out_rowptr[o];
        oe[j] = g.out_rowptr[o + 1];
    }
    constexpr int kAtOnce = 4;
#pragma unroll
    for (int j0 = 0; j0 < kBandPer; j0 += kAtOnce) {
        int32_t t[kAtOnce][4];
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) t[j][k] = g.in_idx[min(rec[j0 + j].x + k, g.nnz_in - 1)];
#pragma unroll
        for (int j = 0; j < kAtOnce; ++j) {
            const int at = (j0 + j) * kBandPlanThreads + tid, i = min(at, n - 1);
            const int32_t o = lo + i, b = ob[j0 + j], e = oe[j0 + j], z = b + shift;
            const int4 r = rec[j0 + j];
            s_out[i] = (uint16_t)(b - first_out);           // (the same value from every thread that writes one)
            if (i == n - 1) s_out[n] = (uint16_t)(e - first_out);
            bad |= e > b && (r.w != e - b || r.z != z);
            bad |= e - first_out > 65535 || e - b > kBandStepOuts;
            uint32_t slot[4];
            int32_t last = -1;
            auto input = [&](int32_t x) {
                if (x < shift) return;
                bad |= x >= z;
                last = max(last, x);
                dist = max(dist, e + shift - x);
            };
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                slot[k] = kBandNowhere + 2 * (o & (kWave - 1));
                if (k < r.y) {
                    input(t[j][k]);
                    slot[k] = band_slot(t[j][k], shift);
                }
            }
#pragma unroll 1
            for (int k = 4; k < r.y; ++k) input(g.in_idx[r.x + k]);
            if (r.y > 4 || e - b > 2) slot[3] = kBandMore;
            const uint32_t out0 = e > b ? band_slot(z, shift) : kBandZero, out1 = e > b + 1 ? band_slot(z + 1, shift) : out0;
            if (at < n) {
                uint32_t *to = a.entry + (int64_t)o * 3;
                to[0] = out0 | out1 << 16;
                to[1] = slot[0] | slot[1] << 16;
                to[2] = slot[2] | slot[3] << 16;
            }
            newest[j0 + j] = last;
        }
    }
#pragma unroll
    for (int j = 0; j < kBandPer; ++j) newest[j] = newest[j] >= 0 ? producer_of(g, newest[j]) : -1;
#pragma unroll
    for (int j = 0; j < kBandPer; ++j)
        if (j * kBandPlanThreads + tid < n) s_begin[j * kBandPlanThreads + tid] = newest[j];
    __syncthreads();
    // running maximum over the segment: eight operators per thread, then threads, then waves
    int last[kBandPer], run = -1;
#pragma unroll
    for (int j = 0; j < kBandPer; ++j) {
        const int i = tid * kBandPer + j;
        if (i < n) run = max(run, s_begin[i]);
        last[j] = run;
    }
    const int upto = wave_incl_max(run);
    if (lane == kWave - 1) s_wave[wave] = upto;
    int before = __shfl_up(upto, 1, kWave);
    if (lane == 0) before = -1;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before = max(before, s_wave[w]);
#pragma unroll
    for (int j = 0; j < kBandPer; ++j) {
        const int i = tid * kBandPer + j;
        if (i >= n) break;
        // begin of the step [begin, i + 1), within the segment
        int begin = max(max(before, last[j]) + 1 - lo, max(i + 1 - kBandStepOps, 0));
        bad |= begin > i;                                    // (an operator that reads from itself or a later one)
        begin = min(begin, i);
        while (s_out[i + 1] - s_out[begin] > kBandStepOuts && begin < i) ++begin;
        s_begin[i] = begin;
    }
    __syncthreads();
    if (tid == 0) {
        int b = n, k = 0;
        while (b > 0 && k < kBandSegSteps) {
            b = s_begin[b - 1];
            s_list[++k] = b;
        }
        s_list[0] = n;
        s_steps = k;
        if (b > 0) s_bad = 1;
    }
    if (bad) s_bad = 1;
    const int wdist = wave_max(dist);
    if (lane == 0) atomicMax(&s_dist, wdist);
    __syncthreads();
    const int steps = s_steps;
    int span = 0;
    for (int k = tid; k < steps; k += kBandPlanThreads) {
        const int b = s_list[k + 1];
        span = max(span, (int)s_out[s_list[k]] - (int)s_out[b]);
        a.steps[(int64_t)blockIdx.x * kBandSegSteps + k] = make_int2(lo + b, first_out + s_out[b] + shift);
    }
    span = wave_max(span);
    if (lane == 0) atomicMax(&s_span, span);
    __syncthreads();
    if (tid == 0) a.segs[blockIdx.x] = make_int4(steps, s_dist, s_span, s_bad);
}

// ORs the bits of sixteen sets into a slot: either half of an LDS word
__device__ __forceinline__ void band_or(uint32_t *lds, uint32_t slot, uint32_t bits)
{
    (void)__hip_atomic_fetch_or(&lds[slot >> 1], bits << ((slot & 1) * 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <bool kFromM>
__global__ __launch_bounds__(2 * kBandHalf) void k_band_sweep(BandArgs a)
{
    extern __shared__ uint32_t lds[];
    const GraphView &g = a.g;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, slice = blockIdx.x;
    constexpr int N = 2 * kBandHalf;
    const int num_segs = (g.num_ops + kBandSegOps - 1) / kBandSegOps;
    const int32_t t_first = g.num_tensors - g.nnz_out;
    uint16_t *ring = reinterpret_cast<uint16_t *>(lds);
    int *s_first = reinterpret_cast<int *>(lds + kBandStepsAt) + 2 * (kBandMaxSteps + 1 + kBandPad);     // by segment, the highest first: steps of those before
    int &s_dist = s_first[kBandMaxSegs + 1], &s_span = s_first[kBandMaxSegs + 2], &s_bad = s_first[kBandMaxSegs + 3];
    int &s_top = s_first[kBandMaxSegs + 4], &s_skip = s_first[kBandMaxSegs + 5], &s_err = s_first[kBandMaxSegs + 6];
    int32_t *s_row = s_first + kBandMaxSegs + 8;            // row pointers of this workgroup's sets
    int2 *step = reinterpret_cast<int2 *>(lds + kBandStepsAt);               // [i]: step i is operators [step[i + 1].x, step[i].x), tensors by .y
    uint16_t *M = reinterpret_cast<uint16_t *>(a.M) + slice;                 // (4 per mask)
    if (tid == 0) {
        s_dist = s_span = s_bad = s_skip = s_err = 0;
        s_top = -1;
    }
    if (!kFromM && tid <= 16) s_row[tid] = a.tgt_rowptr[min(slice * 16 + tid, a.num_sets)];
    for (int i = tid; i < kBandStepsAt; i += N) lds[i] = 0;
    __syncthreads();
    // steps of all segments, highest operators first; the highest target
    int top = -1;
    for (int64_t j = tid; kFromM && j < a.num_targets; j += N) {
        const int32_t t = a.tgt_idx[j];
        if (t < g.num_tensors) top = max(top, t);
    }
    if (wave == 0) {
        int sum = 0;
        for (int i = 0; i < num_segs; i += kWave) {
            const int4 v = i + lane < num_segs ? a.segs[num_segs - 1 - i - lane] : make_int4(0, 0, 0, 0);
            const int upto = wave_incl_scan(v.x);
            if (i + lane < num_segs) s_first[i + lane] = sum + upto - v.x;
            sum += __builtin_amdgcn_readlane(upto, kWave - 1);
            const int dist = wave_max(v.y), span = wave_max(v.z), bad = wave_max(v.w);
            if (lane == 0) {
                s_dist = max(s_dist, dist);
                s_span = max(s_span, span);
                s_bad |= bad;
            }
        }
        if (lane == 0) s_first[num_segs] = sum;
    }
    top = wave_max(top);
    if (lane == 0) atomicMax(&s_top, top);
    __syncthreads();
    const int n = s_first[num_segs];
    top = s_top;
    const bool takes = !s_bad && n <= kBandMaxSteps && (n <= kBandFewSteps || (int64_t)n * kBandMeanOps <= g.num_ops) && s_dist + 4 * s_span <= kBandRing;
    if (slice == 0 && tid == 0) {
        a.host_status[kBandTaken] = takes ? n + 1 : 0;
        if (!takes) atomicOr(&a.state->error, kErrOverflow);                 // (whatever the compaction makes of this is not kept)
    }
    if (!takes) return;
    int skip = 0;                                           // steps that lie above every target
    for (int i = wave; i < num_segs; i += N / kWave) {
        const int at = s_first[i], count = s_first[i + 1] - at;
        for (int k = lane; k < count; k += kWave) {
            const int2 v = a.steps[(int64_t)(num_segs - 1 - i) * kBandSegSteps + k];
            step[at + k + 1] = v;
            skip += v.y > top;
        }
    }
    skip = wave_sum(skip);
    if (kFromM && lane == 0) atomicAdd(&s_skip, skip);
    if (!kFromM && tid == 0) s_skip = n;
    if (tid == 0) step[0] = make_int2(g.num_ops, g.num_tensors);
    if (tid < kBandPad) step[n + 1 + tid] = make_int2(0, t_first);
    if (kFromM)
        for (int t = tid; t < t_first; t += N) ring[kBandRing + t] = M[(int64_t)t * 4];
    __syncthreads();
    // Targets (the threads of the tensors' half hold them): the step that writes them, slot and set
    int target_step[kBandHeld];
    uint32_t target[kBandHeld];
    if (!kFromM) {
        const int64_t j0 = max(s_row[0], 0), j1 = min((int64_t)s_row[16], a.num_targets);
        int err = 0, first = n;
#pragma unroll
        for (int h = 0; h < kBandHeld; ++h) {
            target_step[h] = -1;
            target[h] = 0;
            const int64_t j = j0 + h * kBandHalf + tid - kBandHalf;
            if (tid < kBandHalf || j >= j1) continue;
            int q = 0;
            while (q < 15 && s_row[q + 1] <= j) ++q;
            if (!(s_row[q] <= j && j < s_row[q + 1])) continue;              // (an entry that belongs to no set)
            const int32_t t = a.tgt_idx[j];
            if (t < 0 || t >= g.num_tensors) {
                err = kErrIdRange;
                continue;
            }
            const uint32_t slot = band_slot(t, t_first);
            if (t < t_first) {
                band_or(lds, slot, 1u << q);
                continue;
            }
            int lo = 0, hi = n;                             // the step [lo, hi) that writes t: step[hi].y <= t < step[lo].y
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (step[mid].y <= t) hi = mid; else lo = mid;
            }
            target_step[h] = lo;
            target[h] = slot | (uint32_t)q << 16;
            first = min(first, lo);
        }
        if (err) atomicOr(&s_err, err);
        first = -wave_max(-first);
        if (lane == 0) atomicMin(&s_skip, first);
        __syncthreads();
        if (tid == 0) {
            a.host_status[kBandErrors + slice] = s_err;
            if (s_err) atomicOr(&a.state->error, s_err);
        }
    } else if (slice == 0 && tid == 0) {
        a.host_status[kBandErrors] = a.state->error;
    }
    const int s0 = s_skip;
    auto barrier = [&]() {                                  // (LDS alone: loads and stores stay in flight)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // Both halves run whole rounds of kBandAhead steps (behind the last one empty ones), and every step has the same loads in
    // every lane, so that the compiler knows how many are in flight: what a lane does not have lies past the end of a
    // buffer, where loads give 0 and stores do nothing.  A step's bounds are scalars, read from LDS a step before they are needed.
    auto bound = [&](int i, bool tensor) { return tensor ? step[i].y : step[i].x; };
    const int my_first = (__builtin_amdgcn_readfirstlane(wave) & (kBandHalf / kWave - 1)) * kWave;       // this wave's operators or tensors in a step
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    if (tid < kBandHalf) {
        // operators
        const auto entries = __builtin_amdgcn_make_buffer_rsrc(a.entry, 0, g.num_ops * kEntryBytes, kBufferWord);
        Entry entry[kBandAhead];
        auto fetch = [&](int32_t from) -> Entry {
            return __builtin_amdgcn_raw_buffer_load_b96(entries, tid * kEntryBytes, from * kEntryBytes, 0);
        };
#pragma unroll
        for (int u = 0; u < kBandAhead; ++u) entry[u] = fetch(uniform(bound(s0 + u + 1, false)));
        int32_t end = uniform(bound(s0, false)), from = uniform(bound(s0 + 1, false)), ahead = uniform(bound(s0 + kBandAhead + 1, false));
        barrier();                                          // target bits of the first two steps are in place
        for (int i0 = s0; i0 < n; i0 += kBandAhead) {
#pragma unroll
            for (int u = 0; u < kBandAhead; ++u) {
                Entry e = entry[u];
                const int32_t next_from = bound(i0 + u + 2, false), next_ahead = bound(i0 + u + kBandAhead + 2, false);
                const bool valid = tid < end - from;
                uint32_t k = 0;
                if (from + my_first < end) {                // (some operator is this wave's; the others read what they may not use)
                    k = (uint32_t)ring[e.x & 0xffff] | ring[e.x >> 16];
                    k = valid ? k : 0;
                    if (__builtin_expect(valid && e.z >> 16 == kBandMore, 0)) {
                        const int4 rec = op_record(g, from + tid);
#pragma unroll 1
                        for (int j = 2; j < rec.w; ++j) k |= ring[band_slot(rec.z + j, t_first)];
                        if (k)
#pragma unroll 1
                            for (int j = 3; j < rec.y; ++j) band_or(lds, band_slot(g.in_idx[rec.x + j], t_first), k);
                        e.z = (e.z & 0xffff) | (uint32_t)(kBandNowhere + 2 * lane) << 16;
                    }
                    if (k) {
                        band_or(lds, e.y & 0xffff, k);
                        band_or(lds, e.y >> 16, k);
                        band_or(lds, e.z & 0xffff, k);
                        band_or(lds, e.z >> 16, k);
                    }
                }
                entry[u] = fetch(ahead);
                end = from;
                from = uniform(next_from);
                ahead = uniform(next_ahead);
                barrier();
            }
        }
    } else {
        // tensors
        const int at = tid - kBandHalf;
        const auto masks = __builtin_amdgcn_make_buffer_rsrc(a.M, 0, g.num_tensors * (int)sizeof(u64), kBufferWord);
        uint16_t seed[kBandAhead][2] = {};
        // slot of tensor from + lane's place: at most once around the ring
        auto slot_of = [&](int32_t from, int place) {
            const uint32_t s = (uint32_t)from % (uint32_t)kBandRing + (uint32_t)place;
            return min(s, s - (uint32_t)kBandRing);
        };
        auto fetch = [&](int32_t from, uint16_t (&to)[2]) {
#pragma unroll
            for (int h = 0; h < 2 && kFromM; ++h)
                to[h] = __builtin_amdgcn_raw_buffer_load_b16(masks, (at + h * kBandHalf) * 8, from * 8 + slice * 2, 0);
        };
        int next_target = 0x7fffffff;                       // the next step that one of the wave's targets is for
        if (!kFromM) {
            int first = -0x7fffffff;
#pragma unroll
            for (int h = 0; h < kBandHeld; ++h)
                if (target_step[h] >= 0) first = max(first, -target_step[h]);
            next_target = -wave_max(first);
        }
        auto place = [&](int i, int32_t from, int32_t end, const uint16_t (&bits)[2]) {
            if (kFromM) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (at + h * kBandHalf < end - from && bits[h]) band_or(lds, slot_of(from, at + h * kBandHalf), bits[h]);
            } else if (i == next_target) {                  // uniform
                int later = -0x7fffffff;
#pragma unroll
                for (int h = 0; h < kBandHeld; ++h) {
                    if (target_step[h] == i) band_or(lds, target[h] & 0xffff, 1u << (target[h] >> 16));
                    if (target_step[h] > i) later = max(later, -target_step[h]);
                }
                next_target = -wave_max(later);
            }
        };
        // M of a step's tensors.  A wave's instructions here are what a step waits for, branches above
        // all (reads in one step and stores in the next: 160 -> 193 us for 500 layers of 400).
        auto around = [](uint32_t slot) { return min(slot, slot - (uint32_t)kBandRing); };
        auto flush = [&](int32_t from, int tensors, uint32_t from_slot) {
            if (my_first >= tensors) return;                // uniform
            const uint32_t slot = at < tensors ? around(from_slot + at) : kBandNowhere + 2 * lane;
            const uint32_t m = ring[slot];
            if (my_first + kBandHalf < tensors) {
                const bool is = at + kBandHalf < tensors;
                const uint32_t slot1 = is ? around(from_slot + at + kBandHalf) : kBandNowhere + 2 * lane + 1;
                const uint32_t m1 = ring[slot1];
                ring[slot1] = 0;
                __builtin_amdgcn_raw_buffer_store_b16((unsigned short)m1, masks, is ? (at + kBandHalf) * 8 : kPastEnd, from * 8 + slice * 2, 0);
            }
            ring[slot] = 0;
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)m, masks, at < tensors ? at * 8 : kPastEnd, from * 8 + slice * 2, 0);
        };
        int32_t y0 = uniform(bound(s0, true)), y1 = uniform(bound(s0 + 1, true)), y2 = uniform(bound(s0 + 2, true));
        {
            uint16_t early[2][2] = {};
            fetch(y1, early[0]);
            fetch(y2, early[1]);
            place(s0, y1, y0, early[0]);
            place(s0 + 1, y2, y1, early[1]);
        }
#pragma unroll
        for (int u = 0; u < kBandAhead; ++u) fetch(uniform(bound(s0 + u + 3, true)), seed[u]);
        // of the step before (none yet): first tensor, how many, slot; [place_from, place_end): two steps ahead
        int32_t flush_from = y0, place_end = y2, place_from = uniform(bound(s0 + 3, true)),
                ahead = uniform(bound(s0 + kBandAhead + 3, true));
        int tensors = 0;
        uint32_t flush_slot = (uint32_t)y0 % (uint32_t)kBandRing;
        barrier();
        auto one = [&](int i, uint16_t (&bits)[2]) {
            const int32_t next = bound(i + 1, true);
            const int32_t next_place = kFromM ? bound(i + 4, true) : 0, next_ahead = kFromM ? bound(i + kBandAhead + 4, true) : 0;
            flush(flush_from, tensors, flush_slot);
            place(i + 2, place_from, place_end, bits);
            if (kFromM) {
                fetch(ahead, bits);
                place_end = place_from;
                place_from = uniform(next_place);
                ahead = uniform(next_ahead);
            }
            const int32_t y = uniform(next);
            tensors = flush_from - y;
            flush_from = y;
            flush_slot -= (uint32_t)tensors;                // (below zero: past the highest number)
            flush_slot = min(flush_slot, flush_slot + (uint32_t)kBandRing);
            // What this step has stored, zeros and the target bits of two steps ahead, must be in place at this wave's next barrier, not at this one.
            // LDS operations of a wave complete in order, so that it is enough if a read that follows the stores of the step before has
            // arrived here: `next`.  The asm takes it, which keeps the wait for it in front of the barrier.  (As compiled it is a wait for all of
            // them, or with target bits from M for all but one: branches with and without stores meet here.)
            asm volatile("; bound of the next step: %0" :: "s"(y) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        for (int i0 = s0; i0 < n; i0 += kBandAhead) {
            if (kFromM) {
#pragma unroll
                for (int u = 0; u < kBandAhead; ++u) one(i0 + u, seed[u]);
            } else {                                        // (no loads: the less code the better)
#pragma unroll 1
                for (int u = 0; u < kBandAhead; ++u) one(i0 + u, seed[0]);
            }
        }
        flush(flush_from, tensors, flush_slot);
    }
    __syncthreads();
    for (int t = tid; t < t_first; t += N) M[(int64_t)t * 4] = ring[kBandRing + t];
}

size_t band_scratch(BandArgs &a, void *mem)
{
    char *p = static_cast<char *>(mem);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += (bytes + 255) & ~(size_t)255;
        return r;
    };
    const size_t segs = ((size_t)a.g.num_ops + kBandSegOps - 1) / kBandSegOps;
    a.entry = reinterpret_cast<uint32_t *>(take((size_t)a.g.num_ops * kEntryBytes));
    a.steps = reinterpret_cast<int2 *>(take(segs * kBandSegSteps * sizeof(int2)));
    a.segs = reinterpret_cast<Quad *>(take(segs * sizeof(int4)));
    return off;
}

hipError_t launch_band_plan(const BandArgs &a, int num_cus, hipStream_t s)
{
    const unsigned segs = (unsigned)((a.g.num_ops + kBandSegOps - 1) / kBandSegOps);
    hipLaunchKernelGGL(k_band_plan, dim3(segs + (unsigned)num_cus), dim3(kBandPlanThreads), 0, s, a);
    return hipGetLastError();
}

template <bool kFromM> static hipError_t launch_sweep(const BandArgs &a, hipStream_t s)
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_band_sweep<kFromM>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBandLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_band_sweep<kFromM>, dim3((unsigned)((a.num_sets + 15) / 16)), dim3(2 * kBandHalf), kBandLds, s, a);
    return hipGetLastError();
}

hipError_t launch_band_sweep(const BandArgs &a, bool from_m, hipStream_t s)
{
    return from_m ? launch_sweep<true>(a, s) : launch_sweep<false>(a, s);
}

}  // namespace dgn
