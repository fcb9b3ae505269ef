// Internal declarations shared by the translation units of libdgn (gfx950, wave64 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dgn.h"

typedef unsigned long long u64;   // matches the operand type of HIP's 64-bit atomics
static_assert(sizeof(u64) == sizeof(uint64_t), "u64 must be 64 bits");

namespace dgn {

constexpr int kWave = 64;

// Sticky device-side error bits (TravState::error, BuildStatus::error).
enum : int32_t {
    kErrIdRange = 1,      // operator / tensor / target id out of range
    kErrTopo = 2,         // producer id >= consumer id
    kErrCsr = 4,          // row pointers not monotone / not ending at nnz
    kErrCrossGraph = 8,   // target or edge outside its own packed graph
    kErrOverflow = 16,    // internal: a frontier queue overflowed, the fix-up sweep must run
    kErrLogFull = 32,     // internal: the log of coloured tensors overflowed, the next prune clears everything
};

// Sixteen bytes in memory of the caller, who is asked for eight bytes of alignment.
typedef int4 Quad __attribute__((aligned(8)));
typedef uint4 UQuad __attribute__((aligned(8)));

// Adjacency of a built graph as the kernels see it (device pointers).
struct GraphView {
    int32_t num_ops, num_tensors;
    int32_t nnz_in, nnz_out;
    int32_t num_graphs;
    const int32_t *in_rowptr, *in_idx;
    const int32_t *out_rowptr, *out_idx;
    const int32_t *prod_rowptr, *prod_idx;
    const int64_t *op_off, *t_off;    // [G+1] device copies, NULL when num_graphs == 1
    // What the traversal reads per operator and per pushed tensor (see traverse.hip).  Of graphs whose outputs are one run of tensors
    // (run_shift >= 0) it follows from the adjacency, and these two are not written.
    const Quad *orec;                 // [P] operator record (first input edge, fan-in, outputs); NULL: by rows and ofirst
    const int32_t *ofirst;            // [P] batches that are swept (is_swept in api.hip): the first output, if an operator's outputs are consecutive, else -1
    const int32_t *prod1;             // [T] the producer of a tensor, or kMulti / kNoProducer
    // >= 0: the outputs of operator o are the tensors out_rowptr[o] + run_shift .. out_rowptr[o + 1] + run_shift - 1 (in any order
    // inside its row), each written by nobody else, so that tensor t is written by prod_idx[t - run_shift]; -1: not so
    int32_t run_shift;
};

// Operator record: x = first entry of the operator's row in in_idx, y = its fan-in, and the outputs: w >= 0
// says that the operator writes the w tensors z, z + 1, ... (consecutive ids in the order of its row, the usual
// case for a graph whose tensors are numbered as they are created), w < 0 that its -w outputs are
// out_idx[z], out_idx[z + 1], ...
// prod1 values below zero:
constexpr int32_t kMulti = -2;        // several producers: see prod_rowptr / prod_idx
constexpr int32_t kNoProducer = -3;   // graph input

// The record of operator o and the producer word of tensor t.  Graphs in one run have neither in memory: their rows say the same, and
// not writing them spares a build of 50 M operators 1.6 of 5.6 GB (1 183 -> 845 us); a record then is two accesses of 8 bytes
// in two arrays, so two lines, instead of one of 16.  The traversal's kernels are told which it is (a branch there costs them 7 %).
typedef int IntPair __attribute__((ext_vector_type(2), aligned(4)));
enum RowForm : int { kRecords, kRun, kFirst };     // what an operator's record and a tensor's producer are taken from
__host__ __device__ inline RowForm rows_of(const GraphView &g) { return g.run_shift >= 0 ? kRun : g.orec ? kRecords : kFirst; }
template <RowForm kForm> __device__ __forceinline__ int4 op_record(const GraphView &g, int32_t o)
{
    if (kForm == kRecords) return g.orec[o];
    const int32_t first = kForm == kFirst ? g.ofirst[o] : 0;
    const IntPair in = *reinterpret_cast<const IntPair *>(g.in_rowptr + o), out = *reinterpret_cast<const IntPair *>(g.out_rowptr + o);
    if (kForm == kRun) return make_int4(in.x, in.y - in.x, out.x + g.run_shift, out.y - out.x);
    return make_int4(in.x, in.y - in.x, first >= 0 ? first : out.x, first >= 0 ? out.y - out.x : out.x - out.y);
}
template <RowForm kForm> __device__ __forceinline__ int32_t producer_of(const GraphView &g, int32_t t)
{
    if (kForm != kRun) return g.prod1[t];
    return t >= g.run_shift ? g.prod_idx[t - g.run_shift] : kNoProducer;
}
__device__ __forceinline__ int4 op_record(const GraphView &g, int32_t o)
{
    const RowForm rows = rows_of(g);
    return rows == kRun ? op_record<kRun>(g, o) : rows == kRecords ? op_record<kRecords>(g, o) : op_record<kFirst>(g, o);
}
__device__ __forceinline__ int32_t producer_of(const GraphView &g, int32_t t)
{
    return g.run_shift >= 0 ? producer_of<kRun>(g, t) : producer_of<kRecords>(g, t);
}

// Record of one launch of the traversal: the state it started from and whether it ran a level.
// Launch e writes record e & 1 (one thread, at its start) and reads record (e - 1) & 1, which nobody
// writes while launch e runs.  No block ever waits for another: a launch leaves raw tallies behind
// (push counters, expansion counts, largest deferred operator id, all spread over 64 words), and EVERY
// block of the next launch derives the next state from the previous record and those tallies by itself.
struct LevelSlot {
    int32_t level;          // levels completed before this launch; queue parity = level & 1
    int32_t n;              // entries in the frontier this launch started from
    int32_t theta;          // entries whose producer id is below this are deferred at this level
    int32_t theta_hi;       // deferred operators with id in [theta, theta_hi) are expanded at this level
    int32_t deferred_seen;  // some operator has been deferred so far
    int32_t worked;         // the launch ran a level: its tallies still have to be folded into the state
    int32_t max_key1;       // 1 + largest operator id deferred so far (0: none)
    int32_t pad;
};

constexpr int kMaxRuns = 4;
struct TravState {            // header of the traversal state; the host reads these 128 bytes back
    LevelSlot slot[2];
    int32_t error;             // sticky kErr* bits
    int32_t pad0;
    u64 tensor_visits;         // expansions, summed over levels
    u64 max_frontier;
    int32_t changed;           // fix-up sweep: some operator gained bits
    int32_t run_len;           // wide levels run since the frontier was last small enough for one workgroup
    int32_t n_runs;            // such stretches completed so far; the first kMaxRuns lengths are kept
    int32_t wide_runs[kMaxRuns];
    int32_t pad;
    u64 atomic_updates;        // atomic ORs on M and K issued so far (one per input edge of an operator that gained bits)
};

// Contended words live 64 bytes apart, one per queue segment / block group.
constexpr int kMaxSeg = 64;
// Optional per-level trace (frontier size, expansions, threshold, range top), first kTraceLevels levels.
constexpr int kTraceLevels = 4096;
struct SegCounter {
    int32_t v;           // pushes into this segment of the frontier the launch produced (or handed on)
    int32_t key1;        // 1 + largest operator id deferred by the workgroups that tally here
    int32_t proc;        // entries / operators expanded by those workgroups ...
    int32_t atomics;     // ... and the atomic ORs on M and K they issued (the two are added as one 64-bit word)
    int32_t pad[12];
};
// Tallies of a launch, in buffer (launch number) % 3: written by launch e, read by launch e + 1, zeroed by
// launch e + 2 (one wave, at its start) for launch e + 3.
struct TravCounters { SegCounter cnt[3][kMaxSeg]; };
// Deferral schedule: the threshold starts at theta0, is multiplied by decay after every wide level and
// drops to 0 (nothing deferred any more) once it falls below theta_floor.
struct Schedule { float decay; int32_t theta0; int32_t theta_floor; int32_t small_level; };
// A frontier queue: S segments (power of two, <= kMaxSeg) of seg_cap entries each.
struct QueueGeom { int32_t S; int32_t seg_cap; };
static_assert(sizeof(TravState) == 128, "TravState is read back as 128 bytes");

// Log of the tensors a prune coloured (each exactly once, when its mask left zero), in kMaxSeg segments of
// seg_cap ids with one counter each.  entries == nullptr: no log is kept.
struct ColourLog { int32_t *entries; SegCounter *cnt; int32_t seg_cap; };
// What a prune that kept a complete log leaves in its scratch buffer: which buffers hold its result.  A later
// prune that finds exactly this there zeroes only what the log and the kept list name.
struct RecycleHeader {
    u64 magic, graph_serial;
    const void *M, *K, *kept_ops, *kept_count, *flags;
    const void *also_M, *also_K;   // two more arrays that hold non-zero words only where M / K do (or NULL)
    u64 pad[3];
};
__device__ __forceinline__ bool same_header(const RecycleHeader &a, const RecycleHeader &b)
{
    return a.magic == b.magic && a.graph_serial == b.graph_serial && a.M == b.M && a.K == b.K &&
           a.kept_ops == b.kept_ops && a.kept_count == b.kept_count && a.flags == b.flags && a.also_M == b.also_M &&
           a.also_K == b.also_K;
}

// ---- wave64 helpers ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }
__device__ __forceinline__ u64 lanemask_lt() { return ((u64)1 << lane_id()) - 1; }
__device__ __forceinline__ u64 ballot64(bool p) { return __ballot(p); }
// acc | (a ^ b) in one instruction (a three-input bit operation with the truth table 0xF0 | (0xCC ^ 0xAA))
__device__ __forceinline__ uint32_t or_of_xor(uint32_t acc, uint32_t a, uint32_t b)
{
    return __builtin_amdgcn_bitop3_b32(acc, a, b, 0xF6);
}

// Scans and reductions over the 64 lanes by data-parallel-primitive moves (shifts inside a row of 16 lanes, then a
// broadcast of lane 15 of a row to the next row and of lane 31 to the upper half): eight cheap vector instructions
// where a shuffle-based scan is six cross-lane permutes, each with the latency of an LDS access.
//   kRowShr + n: lane i of a row reads lane i - n of its row (lanes without a source keep `identity`);
//   kRowBcast15 / kRowBcast31 with row masks 0xa / 0xc: rows 1 and 3 read lane 15 of the row before, rows 2 and 3
//   read lane 31.
constexpr int kRowShr = 0x110, kRowBcast15 = 0x142, kRowBcast31 = 0x143;

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_move(int identity, int v)
{
    return __builtin_amdgcn_update_dpp(identity, v, CTRL, ROW_MASK, 0xf, false);
}

__device__ __forceinline__ int wave_incl_scan(int v)
{
    v += dpp_move<kRowShr + 1, 0xf>(0, v);
    v += dpp_move<kRowShr + 2, 0xf>(0, v);
    v += dpp_move<kRowShr + 4, 0xf>(0, v);
    v += dpp_move<kRowShr + 8, 0xf>(0, v);
    v += dpp_move<kRowBcast15, 0xa>(0, v);
    v += dpp_move<kRowBcast31, 0xc>(0, v);
    return v;
}
// inclusive running maximum
__device__ __forceinline__ int wave_incl_max(int v)
{
    constexpr int kLowest = -2147483647 - 1;
    v = max(v, dpp_move<kRowShr + 1, 0xf>(kLowest, v));
    v = max(v, dpp_move<kRowShr + 2, 0xf>(kLowest, v));
    v = max(v, dpp_move<kRowShr + 4, 0xf>(kLowest, v));
    v = max(v, dpp_move<kRowShr + 8, 0xf>(kLowest, v));
    v = max(v, dpp_move<kRowBcast15, 0xa>(kLowest, v));
    v = max(v, dpp_move<kRowBcast31, 0xc>(kLowest, v));
    return v;
}
__device__ __forceinline__ int wave_incl_or(int v)
{
    v |= dpp_move<kRowShr + 1, 0xf>(0, v);
    v |= dpp_move<kRowShr + 2, 0xf>(0, v);
    v |= dpp_move<kRowShr + 4, 0xf>(0, v);
    v |= dpp_move<kRowShr + 8, 0xf>(0, v);
    v |= dpp_move<kRowBcast15, 0xa>(0, v);
    v |= dpp_move<kRowBcast31, 0xc>(0, v);
    return v;
}
// reductions: the last lane of the scan holds the result (one scalar read)
__device__ __forceinline__ int wave_max(int v) { return __builtin_amdgcn_readlane(wave_incl_max(v), kWave - 1); }
__device__ __forceinline__ int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_incl_scan(v), kWave - 1); }
__device__ __forceinline__ u64 wave_or(u64 v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(wave_incl_or((int)(uint32_t)v), kWave - 1);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(wave_incl_or((int)(uint32_t)(v >> 32)), kWave - 1);
    return ((u64)hi << 32) | lo;
}
__device__ __forceinline__ u64 shfl64(u64 v, int src) { return (u64)__shfl((long long)v, src, kWave); }
__device__ __forceinline__ u64 shfl_xor64(u64 v, int mask) { return (u64)__shfl_xor((long long)v, mask, kWave); }

// Lanes hold 64-bit rows of a 64x64 bit matrix (row = lane); returns its transpose (lane q receives
// bit q of every lane's word, bit i coming from lane i).  Six butterfly steps.
template <int J>
__device__ __forceinline__ u64 transpose_step(u64 x, u64 lo_mask /* bit positions whose index has bit J clear */)
{
    const u64 other = (u64)__shfl_xor((long long)x, J, kWave);
    return (lane_id() & J) == 0 ? (x & lo_mask) | ((other & lo_mask) << J)
                                : (x & ~lo_mask) | ((other & ~lo_mask) >> J);
}
__device__ __forceinline__ u64 wave_transpose64(u64 x)
{
    x = transpose_step<32>(x, 0x00000000ffffffffull);
    x = transpose_step<16>(x, 0x0000ffff0000ffffull);
    x = transpose_step<8>(x, 0x00ff00ff00ff00ffull);
    x = transpose_step<4>(x, 0x0f0f0f0f0f0f0f0full);
    x = transpose_step<2>(x, 0x3333333333333333ull);
    x = transpose_step<1>(x, 0x5555555555555555ull);
    return x;
}

// Loads that must observe atomics performed by other workgroups / earlier levels: go to the
// device-coherent level instead of a possibly stale per-CU cache line.
__device__ __forceinline__ u64 load_coherent(const u64 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t load_coherent(const int32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Stores that other workgroups read within the same kernel: written through to the device-coherent level.
__device__ __forceinline__ void store_coherent(int32_t *p, int32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(u64 *p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_coherent(uint8_t *p, uint8_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t load_coherent(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sixteen bytes of a stream that nobody reads before the caches have lost it: past them where `stream`.  On streams
// larger than the last-level cache (256 MB) such stores are 8 to 10 % faster; what fits in it is better left there for the
// next kernel.
typedef int Int4Vec __attribute__((ext_vector_type(4), aligned(8)));
constexpr size_t kStreamBytes = (size_t)256 << 20;
template <bool stream> __device__ __forceinline__ void store16(void *p, int a, int b, int c, int d)
{
    const Int4Vec v = {a, b, c, d};
    if (stream) __builtin_nontemporal_store(v, reinterpret_cast<Int4Vec *>(p));
    else *reinterpret_cast<Int4Vec *>(p) = v;
}

// ---- launch wrappers (each returns a hipError_t; nothing synchronises) -------------------------
struct FillRegion { void *ptr; size_t bytes; };   // ptr 8-byte aligned, bytes multiple of 8
hipError_t launch_clear(const FillRegion *regions, int num_regions, hipStream_t s);
// Zero `regions` (at most 8) -- unless *hdr equals `want`: then zero only M of the logged tensors and K and the
// deferral marker of the kept operators (the buffers are as the prune that wrote the header left them), and
// the same words of want.also_M / want.also_K where those are given.
// found_out[0] = 1 when the header was found, else 0.
hipError_t launch_clear_or_reset(const FillRegion *regions, int num_regions, const RecycleHeader *hdr,
                                 const RecycleHeader &want, u64 *found_out, const ColourLog &log, const int32_t *kept_ops,
                                 const int64_t *kept_count, u64 *M, u64 *K, uint8_t *DB, uint8_t *flags, hipStream_t s);

// out[i] = sum_{j<i} in[j], i = 0..n (n+1 outputs; out[n] = total).  in/out may alias when `in`
// holds n+1 entries.  tmp: scratch of scan_tmp_bytes(n) bytes.
size_t scan_tmp_bytes(int64_t n);
hipError_t launch_exclusive_scan(const int32_t *in, int32_t *out, int64_t n, void *tmp, hipStream_t s);

// Stable LSD radix sort of (key, val) pairs on the low `key_bits` bits of the keys.
// Result: vals_out and keys_out.  keys_in / vals_in are not modified.
// tmp: scratch of sort_tmp_bytes(n) bytes.
size_t sort_tmp_bytes(int64_t n);
hipError_t launch_sort_pairs(const int32_t *keys_in, const int32_t *vals_in, int32_t *keys_out,
                             int32_t *vals_out, int64_t n, int key_bits, void *tmp, hipStream_t s);

// rows lo..hi get val; gaps longer than a few rows are filled by the whole wave (call wave-uniformly)
__device__ __forceinline__ void write_rows(int32_t *rowptr, int lo, int hi, int32_t val)
{
    constexpr int kShort = 4;
    for (int r = lo; r <= hi && r < lo + kShort; ++r) rowptr[r] = val;
    u64 longer = ballot64(hi - lo >= kShort);
    while (longer) {
        const int src = __builtin_ctzll(longer);
        longer &= longer - 1;
        const int s_lo = __shfl(lo, src, kWave) + kShort, s_hi = __shfl(hi, src, kWave);
        const int32_t s_val = __shfl(val, src, kWave);
        for (int r = s_lo + lane_id(); r <= s_hi; r += kWave) rowptr[r] = s_val;
    }
}

// An operator's record, as GraphView::orec describes it
template <bool kStream>
__device__ __forceinline__ void write_record(Quad *p, int32_t ib, int32_t ie, int32_t ob, int32_t oe, int32_t first, bool consecutive)
{
    store16<kStream>(p, ib, ie - ib, consecutive ? first : ob, consecutive ? oe - ob : -(oe - ob));
}

// Status words of a build: [0] error bits, then flags
enum : int {
    kStatusInUnsorted = 1,       // the operators of the input edges decrease somewhere
    kStatusOutUnsorted = 2,      // ... of the output edges
    kStatusProdUnsorted = 3,     // the tensors of the output edges, taken in operator order
    kStatusInGap = 5,            // row pointers with a long run of empty rows, left out
    kStatusOutGap = 6,
    kStatusProdGap = 7,
    kStatusOrder = 8,            // (so many words say whether there is an adjacency; the following describe it)
    kStatusNoRows = 9,           // lists sorted by buckets: ids out of range were found before these were made, there are no rows
    kStatusPending = 10,         // ... rows by tensor that do not follow from the rows by operator
    kStatusBig = 11,             // ... how many of them are large: inputs, outputs, outputs by tensor
    kStatusMulti = 16,           // some tensor has several producers
    kStatusScattered = 17,       // the outputs are not one run of tensors up to the last one, or not in this order inside every row
    kStatusNoRun = 18,           // ... in whatever order inside the rows (see GraphView::run_shift)
    kStatusRing = 20,            // what k_records_and_check finds out for the ring sweep: [0] != 0: outputs are not one run or
                                 // read too early; [1] graph inputs, [2] dist, [3] span64 (maxima)
    kStatusSampled = 24,         // operators whose first input was looked at (their graph's outputs are one run) ...
    kStatusWithin8 = 25,         // ... those that read less than an eighth of their graph back,
    kStatusWithin32 = 26,        // ... a 32nd,
    kStatusWithin192 = 27,       // ... a 192nd,
    kStatusWithin640 = 28,       // ... a 640th,
    kStatusWithin2048 = 29,      // ... a 2 048th
    kStatusReach = 30,           // k_records_and_check: how far below an operator's first output its inputs lie at most
    kStatusSoon = 31,            // sampled operators whose first input was written just before (kSoonTensors)
    kStatusLeaveIn = 32,         // (not read back) a look at some places has found the operators of the input edges,
    kStatusLeaveOut = 33,        // of the output edges in no order: the pass over the lists leaves them
    kStatusEnd = 64,
};
// An edge list and where its adjacency goes.  idx / row == NULL: those are in place already.
struct EdgeList {
    const int32_t *op, *tensor;
    int64_t nnz;
    int32_t num_ops, num_tensors;
    int32_t *idx, *row;                          // rows by operator
    int32_t *prod_idx, *prod_row, *prod1;        // outputs: rows by tensor, producer words
    bool may_run;                                // producer words of tensors where one run up to the last would have them are left out
};
// Rows of a list in no order by way of buckets of 2^row_bits rows: `passes` sorting passes of pass_bits bits bring it into
// buckets, a workgroup of `threads` each does the rest (see radix_sort.hip).  use: that is fewer passes over memory than the sort takes.
struct RowPlan { bool use; int row_bits, passes, pass_bits, threads; int64_t buckets; };
RowPlan plan_rows(int64_t nnz, int64_t rows, int key_bits);
// l.row, l.idx and, with `producers`, the rows by tensor.  kErrIdRange: there are ids out of range; kStatusPending: the rows by
// operator are written, those by tensor are not (the outputs are no run of tensors).  tmp: scratch of sort_tmp_bytes(l.nnz) bytes.
// num_big: a word of the status, zero before.
hipError_t launch_bucket_rows(const RowPlan &p, const EdgeList &l, bool producers, int32_t *num_big, int32_t *status, void *tmp, hipStream_t s);
// kErrIdRange if an edge of the list has an id out of range
hipError_t launch_check_ids(const EdgeList &l, int32_t *status, hipStream_t s);
// clears all status words; long lists that are in no order at a few places already are noted
hipError_t launch_first_look(const EdgeList &in, const EdgeList &out, int32_t *status, hipStream_t s);
// one pass over the input edges (NULL: the outputs only) and the output edges: checks them and, assuming that they are in
// order, writes the finished adjacency
// maybe_left: the outputs' rows by tensor are likely to be there already (kStatusLeaveOut)
hipError_t launch_scan_edges(const EdgeList *in, const EdgeList &out, int32_t *status, hipStream_t s, bool maybe_left = false);
// The kernels from here to launch_check_topological do nothing if the status says that there is no adjacency yet.
// what launch_build_records notes about how far back operators read, where there are no records to be made
hipError_t launch_sample_reach(const GraphView &g, int32_t *status, hipStream_t s);
// operator records (unless the outputs are one run) of a single graph / of graphs that are also checked for range and for the ring
// sweep.  prod1: producer words that the pass over the outputs left out (EdgeList::may_run), or NULL: there are none
hipError_t launch_build_records(const GraphView &g, Quad *orec, int32_t *prod1, int32_t *status, hipStream_t s);
hipError_t launch_records_and_check(const GraphView &g, Quad *orec, int32_t *ofirst, int32_t *prod1, int32_t *status, int num_cus, hipStream_t s);
hipError_t launch_check_topological(const GraphView &g, int32_t *status, hipStream_t s);
// producer words from prod_rowptr / prod_idx; kStatusMulti when some tensor has several producers
hipError_t launch_build_producers(const GraphView &g, int32_t *prod1, int32_t *status, hipStream_t s);
// keys[e] = the tensors of a list in operator order, ascending inside every operator's row; flags rows longer than 64
// (left as they are) as unsorted by tensor, and any change as "scattered"
hipError_t launch_order_rows(const int32_t *ops, const int32_t *tensors, int64_t nnz, int32_t *keys, int32_t *status, hipStream_t s);
// rowptr[0..n_rows] from keys that are in row order; nothing if the status has an error (all are in range)
hipError_t launch_row_bounds(const int32_t *keys, int64_t nnz, int32_t n_rows, int32_t *rowptr, const int32_t *status, hipStream_t s);
hipError_t launch_check_csr(const GraphView &g, int32_t *status, hipStream_t s);
hipError_t launch_expand_rows(const int32_t *rowptr, int32_t n_rows, int32_t nnz, int32_t *row_of, int32_t *run_idx, int32_t *run_row,
                              int32_t num_tensors, int32_t *status, hipStream_t s);

// Traversal.
hipError_t launch_seed(const GraphView &g, int32_t Q, int64_t num_targets, const int32_t *tgt_rowptr,
                       const int32_t *tgt_idx, u64 *M, TravState *st, TravCounters *ctr, int32_t *q0,
                       const QueueGeom &qg, int32_t theta0, const ColourLog &log, hipStream_t s);
// One wide level (whole chip); a frontier of at most narrow_cap entries is left to launch_narrow unless
// deferred operators are waiting.  DB: deferred-operator markers, one byte per operator.
hipError_t launch_level(const GraphView &g, TravState *st, TravCounters *ctr, int launch_no, int32_t *q0, int32_t *q1,
                        const QueueGeom &qg, uint8_t *DB, uint8_t *flags, u64 *M, u64 *K, int grid_blocks, int narrow_cap,
                        const Schedule &sch, const ColourLog &log, Quad *trace, hipStream_t s);
// One workgroup runs level after level while 0 < frontier <= narrow_cap and nothing is deferred.  It leaves no
// tallies behind, so the record it writes is the state the host may read.
hipError_t launch_narrow(const GraphView &g, TravState *st, TravCounters *ctr, int launch_no, int32_t *q0, int32_t *q1,
                         const QueueGeom &qg, uint8_t *DB, uint8_t *flags, u64 *M, u64 *K, int narrow_cap, const Schedule &sch,
                         const ColourLog &log, Quad *trace, hipStream_t s);
// Packed batches of small graphs whose operator ids are a topological order: one wave per graph sweeps
// its operators once, highest ids first (no frontier at all); fills K and, when pq is not NULL, the
// per-graph per-set counts.
hipError_t launch_sweep_graphs(const GraphView &g, u64 *M, u64 *K, int64_t *per_query_count, bool multi_producer,
                               hipStream_t s);
// The same for graphs whose tensors are numbered as they are created and read soon after (see ring_sweep.hip): one
// workgroup per graph, M of the recent tensors in LDS.  Everything is written in full; nothing needs clearing.
constexpr size_t kRingMaxLds = 160 * 1024 - 1024;   // LDS of a compute unit less the kernel's own few words
struct RingArgs {
    GraphView g;
    int32_t num_sets;        // per graph; of a single graph any number, 64 to a word
    int32_t words;           // single graph: words of 64 sets; every output array has a row per word
    int64_t num_targets;
    const int32_t *tgt_rowptr, *tgt_idx;
    u64 *M, *K;
    uint8_t *flags;          // a byte per operator: K != 0, or NULL
    uint8_t *flags2;         // the same once more, or NULL
    int32_t *kept_ops;
    u64 *kept_masks;         // may be NULL
    int64_t *kept_count;
    int64_t *pq;             // [G * 64], may be NULL
    u64 *bits;               // [ring_bit_words(P, G)], per word of sets: a bit per operator, K != 0: words of 64 operators of one graph, graph g's
                             // from entry g + (its first operator) / 64 on
    int32_t *cum;            // for every such word: operators of the graph kept in it and above
    Quad *graphs;            // [G + 1], or [words]: per graph or word of sets: operators kept, error bits, settling steps; all graphs
    int32_t *host_status;    // pinned host memory: error bits, settling steps
    RecycleHeader *hdr, want;
    int32_t recycle;         // *hdr may say that the buffers hold this kernel's last result
    int32_t list_here;       // the sweep makes the ordered list itself
    int32_t ring_words, low_words, seed_words;     // LDS: ring, graph inputs (8 bytes each), targets (4 bytes each)
    // graphs swept in segments (segs > 1): each of them seg_words = 1 << seg_shift words of 64 operators
    int32_t segs, seg_words, seg_shift;
    int32_t few_segs;        // so few that each has kRingPlaceWaves waves to put its targets in place
    int32_t count_steps;     // somebody wants to know the settling steps
    int32_t reach;           // no operator reads a tensor further below its first output (at most kWave)
    u64 *b_M, *b_K;          // [T], [P]: which tensors of the boundary above its segment a tensor or operator is reached from
    u64 *edge;               // [G * segs * (words + 1)][ring_edge_words]: per segment and word: what the boundary below receives, the
                             // graph's inputs, settling steps; the last word: the same in tensors of the boundary above
    u64 *own_bits;           // as bits: operators kept for the segment's own targets
    int32_t *seg_kept;       // [G * segs], batches: operators kept
};
constexpr int kRingExtraWords = 1 + kWave;
__host__ __device__ inline int64_t ring_edge_words(const RingArgs &a) { return kWave + a.low_words + 1; }
constexpr int kRingSegWaves = 1, kRingPlaceWaves = 8;
constexpr int kRingMaxSegs = 1024, kRingMaxSegWords = 256;
// Lays out what segments leave for each other at `mem` (NULL: the bytes alone); g, words, segs and low_words are set
size_t ring_segment_scratch(RingArgs &a, void *mem);
constexpr int64_t kRingMaxGraphOps = (int64_t)1 << 18;   // the largest graph that is ever swept
// words of 64 operators of G graphs, one of them perhaps ragged in each
__host__ __device__ inline int64_t ring_bit_words(int64_t P, int64_t G) { return (P >> 6) + G + 1; }
inline int64_t ring_words(int waves, int dist, int span64)
{
    const int64_t need = (int64_t)dist + 3 * (int64_t)waves * span64;
    int64_t r = 64 * waves;
    while (r < need) r *= 2;
    return r;
}
// ev (or NULL): ev[0] is recorded behind the sweep; with `all`, ev[1] behind the per-graph counts and ev[2] behind the list
hipError_t launch_ring_sweep(RingArgs a, int waves, int dist, int span64, int64_t max_graph_ops, int *launches, hipStream_t s,
                             hipEvent_t *ev, bool all);
// The same for one graph of wide layers (see band_sweep.hip): a workgroup per sixteen sets.  The plan clears M.
constexpr int64_t kBandMaxOps = (int64_t)1 << 20;
constexpr int kBandMaxLow = 8192;         // graph inputs, at most
constexpr int kBandMaxSteps = 4096;
constexpr int kBandStepOps = 512, kBandStepOuts = 1024;
constexpr int64_t kBandMaxTargets = 2048; // that the sweep puts in place itself; more go by way of M and the seed kernel
constexpr int kBandRegions = 6;
enum : int { kBandTaken = 0, kBandFound = 1, kBandErrors = 4 /* by sixteen sets */ };
struct BandArgs {
    GraphView g;
    int32_t num_sets;
    int64_t num_targets;
    const int32_t *tgt_rowptr, *tgt_idx;
    u64 *M;
    TravState *state;        // its error bits
    int32_t *host_status;    // pinned host memory: 1 + steps or 0 (the graph is not of this kind: nothing written), header found, error bits
    RecycleHeader *hdr, want;
    int32_t recycle;
    FillRegion clear[kBandRegions];
    uint32_t *entry;         // [P][3]
    int2 *steps;             // per segment: first operator and tensor of its steps, the highest first
    Quad *segs;              // steps, how far back its operators read, most outputs in a step, not a 0 if unfit
};
size_t band_scratch(BandArgs &a, void *mem);        // lays out the last three (NULL: the bytes alone); g is set
hipError_t launch_band_plan(const BandArgs &a, int num_cus, hipStream_t s);
hipError_t launch_band_sweep(const BandArgs &a, bool from_m, hipStream_t s);
// One sweep over all operators re-deriving K and pushing new bits to the inputs; *changed |= 1 if any.
hipError_t launch_fix_sweep(const GraphView &g, u64 *M, u64 *K, uint8_t *flags, int32_t *changed, int grid_blocks, hipStream_t s);

// Removal rule + compaction.
constexpr int kPqStride = 8;         // int64 words between two replicated per-set counters (64 bytes)
constexpr int kCompactTile = 2048;   // operators per workgroup in the count / scatter passes
struct CompactArgs {
    GraphView g;
    const u64 *M;            // used when from_tensor_mask
    u64 *K;
    uint8_t *op_flag;        // may be NULL
    int32_t *kept_ops;
    u64 *kept_masks;         // may be NULL
    int64_t *kept_count;
    int64_t *per_query_count;   // may be NULL
    int64_t *pq_part;           // [pq_replicas][G*64][kPqStride] zeroed scratch, or NULL: add straight into per_query_count
    int pq_replicas;            // power of two
    u64 *opbits;             // [ceil(P/64)] scratch
    int32_t *block_counts;   // [num_tiles + 1] scratch
    bool from_tensor_mask;   // K := OR M[out] (true) or read K as accumulated by the traversal
    const uint8_t *flag_in;  // when not NULL (and not from_tensor_mask): one byte per operator, 1 where K != 0, as the
                             // traversal left them; K is then read for those operators only
    RecycleHeader *hdr;      // when not NULL: the last pass writes `want` there if no error bit is set in *error
    RecycleHeader want;
    const int32_t *error;
};
// ev (may be NULL): three events recorded after the count, scan and scatter passes.
hipError_t launch_keep_compact(const CompactArgs &a, hipStream_t s, hipEvent_t *ev = nullptr);

// Read-outs of a prune result (Sec. 3.2): ignore mask from the kept list; per-set operator lists.
hipError_t launch_ignore_mask(const GraphView &g, bool several_producers, const int32_t *kept_ops, const u64 *kept_masks, const int64_t *kept_count,
                              const u64 *M, u64 *ignore, int64_t *ignore_count, int grid_blocks, hipStream_t s);
size_t set_lists_scratch_bytes(int64_t num_kept);
hipError_t launch_set_lists(const int32_t *kept_ops, const u64 *kept_masks, int64_t num_kept, int64_t *set_rowptr,
                            int32_t *set_ops, int64_t capacity, void *scratch, int grid_blocks, hipStream_t s);

// Key of a transaction (Sec. 4.1): 128-bit digest of the target sets; *digest_dev points into `scratch`.
constexpr int kDigestMaxBlocks = 1024;
size_t digest_scratch_bytes();
hipError_t launch_target_digest(int32_t num_sets, int64_t n, const int32_t *tgt_rowptr, int64_t num_targets,
                                const int32_t *tgt_idx, void *scratch, u64 **digest_dev, hipStream_t s);

// Backward Prune (Algorithm 2), forward stage: what its passes work on (see backward.hip), by place in the kept list.
struct BackwardLinks {
    u64 *K, *FO;             // [P] K of the first stage; marks that arrive at an operator's inputs
    int2 *group;             // [P / 64 + 1] per 64 kept operators: first entry and number of entries below
    int32_t *link;           // [Ein] the producer of an input, or -1, or -2 - the id of an input with several
    uint8_t *owner;          // [Ein] the operator of the group that reads it
};
BackwardLinks backward_links(void *mem, int64_t P, int64_t Ein, size_t *bytes);
// flags: [0] error bits, [1] cleared with the other 62 and used by the call, [2] ... for the passes
hipError_t launch_link_kept(const GraphView &g, const int32_t *kept, const int64_t *kept_count, u64 *place, const u64 *B, u64 *F,
                            const int32_t *obj, const int32_t *wrt, int num_pairs, const BackwardLinks &b, int32_t *flags,
                            int num_cus, hipStream_t s);
hipError_t launch_forward_pass(const GraphView &g, const int64_t *kept_count, const u64 *place, const BackwardLinks &b,
                               int32_t *changed, int num_cus, hipStream_t s);
hipError_t launch_write_marks(const GraphView &g, bool several_producers, const int32_t *kept, const int64_t *kept_count,
                              const u64 *FO, const u64 *B, u64 *F, u64 *K, uint8_t *flags, int grid_blocks, hipStream_t s);
hipError_t launch_pair_rows(int num_pairs, int32_t *tgt_rowptr, hipStream_t s);     // target row pointers 0..n
hipError_t launch_keep_from_list(const GraphView &g, const int32_t *kept, const int64_t *kept_count, const u64 *F, u64 *K,
                                 uint8_t *flags, int grid_blocks, hipStream_t s);

// In-place structures (Algorithm 3).  counters: [0] = number of nodes in `list`,
// [1 + r] = doubling round r left some jump pointer alive.
constexpr int kInplaceMaxRounds = 32;               // 2^32 links: longer than any chain of int32 ids
struct InplaceBuffers {
    int32_t *child;                                 // the only child of a tensor, -1 none, -2 several
    int32_t *J[2];                                  // jump pointers, double buffered
    int32_t *list;                                  // the nodes that an operator with one output reads (each once)
    int32_t *counters;
};
size_t inplace_scratch_bytes(int64_t T);
InplaceBuffers inplace_buffers(void *scratch, int64_t T);
// init and children (the state before the first doubling round)
// What many operators read at the same time: nothing; the inputs of their graph, in chains (operators that read what was written just before)
// and in packed batches; or nobody knows, where one graph's tensors are not numbered in order.
enum class Meet { nowhere, unknown, chains, batch };
hipError_t launch_inplace_setup(const GraphView &g, const u64 *K, u64 select, const int32_t *kept_ops,
                                const int64_t *kept_count, int32_t *rename, int64_t *renamed_count,
                                const InplaceBuffers &b, Meet meet, int grid_blocks, hipStream_t s);
hipError_t launch_inplace_round(int round, int32_t *rename, int64_t *renamed_count, const InplaceBuffers &b,
                                int grid_blocks, hipStream_t s);

}  // namespace dgn
