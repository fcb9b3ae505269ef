// CSR builder: the pass over the edge lists that checks them and writes the rows, the order of shuffled outputs, row pointers
// of sorted lists, operator records and producer words, and the validation passes.
// The adjacency follows the edge definition of Sec. 2.2 of the paper: an operator with the tensors it
// reads and the tensors it writes; Parent(x) of Algorithm 1 = inputs of every operator that writes x.
#include "common.h"

namespace dgn {

// The rows that position e closes: (prev, cur].  Keys outside their range close none (the call fails anyway), and a
// long run of empty rows is left to a pass of its own (*gap): keys in random order jump far at nearly every position, and
// filling those jumps here would cost more than the sort that follows.  (The rows before a list's first key, often the
// graph's inputs, occur once.)
constexpr int kMaxGapHere = 64;
constexpr int kMaxFirstGap = 8192;
__device__ __forceinline__ void rows_closed(int32_t prev, int32_t cur, int32_t n_rows, int64_t e, int &lo, int &hi, bool &gap)
{
    lo = 0;
    hi = -1;
    if (prev >= -1 && prev < n_rows && cur >= 0 && cur <= n_rows) {
        lo = prev + 1;
        hi = cur;
    }
    if (hi - lo >= (e == 0 ? kMaxFirstGap : kMaxGapHere)) {
        gap = true;
        hi = lo - 1;
    }
}

// One pass over an edge list in the order it was handed over: range check of both ids, whether the keys ever decrease
// (*unsorted = 1), and -- on the assumption that they do not, which holds for a graph recorded operator by operator --
// the finished rows: the operators' row pointers (first position of every operator) and row entries, and for a list of
// outputs also the tensors' (first position of every tensor, producers) and, unless the outputs are one run of tensors up to the last
// (EdgeList::may_run), producer words.  If the keys do decrease
// somewhere, what was written is overwritten by the sort that follows, which also checks every id once more: a wave that has met such a
// place writes nothing.  (The list is read to its end all the same, in pieces handed out in order; of long ones k_first_look sees beforehand whether that
// is worth it.)  No atomic in the common case.
//
// A stream of 12 bytes per input edge and 24 per output edge and tensor: it is bound by memory.  A thread takes four
// neighbouring positions per step, in 16-byte accesses where the arrays are aligned for them (one position per thread left
// the pass waiting for memory).  Outputs take both adjacencies and the producer words from one reading: three passes did
// that before, 0.99 ms of a 50 M-operator graph and 0.3 more for the producer words; then 1.00 in all, with its stores past the
// caches 0.91, without the producer words of one run 0.81, with a workgroup per piece of the lists 0.77 = 5.1 TB/s.
constexpr int kScanThreads = 256, kScanTile = kScanThreads * 4;

template <bool kOut, bool kStream>
__device__ __forceinline__ void scan_list(const EdgeList &l, int64_t block, int64_t blocks, uint32_t *s_words, int32_t *status)
{
    constexpr int kPer = 4;
    const int32_t *ops = l.op, *tensors = l.tensor;
    const int64_t nnz = l.nnz;
    const int32_t P = l.num_ops, T = l.num_tensors;
    const bool copies = l.idx != nullptr;                               // (already in place after a sort)
    uintptr_t all = reinterpret_cast<uintptr_t>(ops) | reinterpret_cast<uintptr_t>(tensors) | reinterpret_cast<uintptr_t>(l.idx);
    if (kOut) all |= reinterpret_cast<uintptr_t>(l.prod_idx);
    const bool wide = (all & 15) == 0;
    const int64_t gsize = blocks * kScanThreads * kPer;
    const int64_t steps = (nnz + 1 + gsize - 1) / gsize;                // position nnz closes the last rows
    const int32_t shift = (int32_t)(T - nnz);                           // outputs in one run: edge e writes tensor e + shift
    bool bad = false, gap = false, tgap = false, multi = false, scattered = false;
    bool down = false, tdown = false;                                   // wave-uniform: operators / tensors decrease somewhere
    for (int64_t st = 0; st < steps; ++st) {                            // whole waves stay in the loop
        const int64_t e0 = st * gsize + (block * kScanThreads + threadIdx.x) * kPer;
        int32_t k[kPer + 1], t[kPer + 2];                               // k[j], t[j]: of position e0 + j - 1
        k[0] = e0 > 0 && e0 <= nnz ? ops[e0 - 1] : -1;
        if (kOut) t[0] = e0 > 0 && e0 <= nnz ? tensors[e0 - 1] : -1;
        const bool inner = wide && e0 + kPer <= nnz;
        if (inner) {
            const int4 kk = *reinterpret_cast<const int4 *>(ops + e0);
            const int4 tt = *reinterpret_cast<const int4 *>(tensors + e0);
            k[1] = kk.x; k[2] = kk.y; k[3] = kk.z; k[4] = kk.w;
            t[1] = tt.x; t[2] = tt.y; t[3] = tt.z; t[4] = tt.w;
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                k[j + 1] = e0 + j < nnz ? ops[e0 + j] : P;
                t[j + 1] = e0 + j < nnz ? tensors[e0 + j] : T;
            }
        }
        if (kOut) t[kPer + 1] = e0 + kPer < nnz ? tensors[e0 + kPer] : T;
        bool d = false, td = false, run = kOut && inner;
#pragma unroll
        for (int j = 1; j <= kPer; ++j) {
            if (e0 + j > nnz) continue;
            if (k[j] < 0 || k[j] >= P || t[j] < 0 || t[j] >= T) bad = true;
            d |= k[j - 1] > k[j];
            if (kOut) {
                td |= t[j - 1] > t[j];
                scattered |= t[j] != (int32_t)(e0 + j - 1) + shift;
                run &= t[j] == t[j - 1] + 1;
            }
        }
        if (kOut) run &= t[kPer + 1] != t[kPer] && t[1] >= 0 && t[kPer] < T;
        down |= ballot64(d) != 0;
        if (down) break;
        if (kOut) tdown |= ballot64(td) != 0;
        if (copies && inner) {
            store16<kStream>(l.idx + e0, t[1], t[2], t[3], t[4]);
        } else if (copies) {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (e0 + j < nnz) l.idx[e0 + j] = t[j + 1];
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            int lo = 0, hi = -1;
            if (l.row && e0 + j <= nnz) rows_closed(k[j], k[j + 1], P, e0 + j, lo, hi, gap);
            write_rows(l.row, lo, hi, (int32_t)(e0 + j));
        }
        if (kOut && !tdown) {
            if (inner) {
                store16<kStream>(l.prod_idx + e0, k[1], k[2], k[3], k[4]);
            } else {
#pragma unroll
                for (int j = 0; j < kPer; ++j)
                    if (e0 + j < nnz) l.prod_idx[e0 + j] = k[j + 1];
            }
            if (run) {                                                  // four new tensors in a row, each with one producer
                int32_t *row = l.prod_row + t[1], *word = l.prod1 + t[1];
                const bool spared = l.may_run && t[1] == (int32_t)e0 + shift;
                if (((reinterpret_cast<uintptr_t>(row) | reinterpret_cast<uintptr_t>(word)) & 15) == 0) {
                    store16<kStream>(row, (int)e0, (int)e0 + 1, (int)e0 + 2, (int)e0 + 3);
                    if (!spared) store16<kStream>(word, k[1], k[2], k[3], k[4]);
                } else {
#pragma unroll
                    for (int j = 0; j < kPer; ++j) {
                        row[j] = (int32_t)e0 + j;
                        if (!spared) word[j] = k[j + 1];
                    }
                }
            }
            if (ballot64(!run) != 0) {
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    int lo = 0, hi = -1;
                    if (!run && e0 + j <= nnz) rows_closed(t[j], t[j + 1], T, e0 + j, lo, hi, tgap);
                    write_rows(l.prod_row, lo, hi, (int32_t)(e0 + j));
                    // producer words: none for the tensors between, and the tensor itself at its first position
                    write_rows(l.prod1, lo, hi - 1, kNoProducer);
                    if (lo <= hi && hi < T) {
                        const bool again = t[j + 2] == hi;
                        l.prod1[hi] = again ? kMulti : k[j + 1];
                        multi |= again;
                    }
                }
            }
        }
    }
    // Shuffled input has every workgroup report: once each, its words looked at together, and a store (same value from everyone)
    // only where it is needed.  (12 M operators in shuffled order, when lists of that length were read here: 125 us with a look at every word
    // by every wave, 59 with one look per workgroup.  3 M, the whole list read: 39.)
    uint32_t words = 0;                                                 // bit w: status word w
    auto report = [&](bool v, int word) { words |= ballot64(v) != 0 ? 1u << word : 0; };
    report(down, kOut ? kStatusOutUnsorted : kStatusInUnsorted);
    report(gap, kOut ? kStatusOutGap : kStatusInGap);
    if (kOut) {
        report(tdown, kStatusProdUnsorted);
        report(tgap, kStatusProdGap);
        report(scattered, kStatusScattered);
        report(scattered, kStatusNoRun);
        report(multi, kStatusMulti);
    }
    if (ballot64(bad) != 0 && lane_id() == 0) atomicOr(status, kErrIdRange);
    if (words == 0) return;                                             // (wave-uniform)
    uint32_t others = 0;                                                // what other waves of the workgroup report
    if (lane_id() == 0) others = atomicOr(s_words, words);
    words &= ~__builtin_amdgcn_readfirstlane(others);
    if (lane_id() < 32 && (words >> lane_id() & 1) && load_coherent(status + lane_id()) == 0) store_coherent(status + lane_id(), 1);
}

// inputs and outputs in one launch; an empty list has one position too (it closes all rows).  leave: what k_first_look has found
template <bool kStream>
__global__ __launch_bounds__(kScanThreads) void k_scan_edges(EdgeList in, EdgeList out, int in_blocks, const int32_t *__restrict__ leave,
                                                             int32_t *__restrict__ status)
{
    __shared__ uint32_t s_words;                                        // status words that some wave reports
    if (leave[(int)blockIdx.x < in_blocks ? 0 : kStatusLeaveOut - kStatusLeaveIn]) return;
    if (threadIdx.x == 0) s_words = 0;
    __syncthreads();
    if ((int)blockIdx.x < in_blocks) scan_list<false, kStream>(in, blockIdx.x, in_blocks, &s_words, status);
    else scan_list<true, kStream>(out, (int)blockIdx.x - in_blocks, (int)gridDim.x - in_blocks, &s_words, status);
}

// A workgroup per 1 024 positions, however many: handed out in order they go through the lists like one long stream.  (8 192 per list, each
// with every 8 192nd piece: 850 us for 50 M operators, 2 048 in all: 975, one each: 797.)  That many would read all of a list in no order before
// the first of them could say so, so that long ones are looked at in a few places before (12 M operators in shuffled order: 1 100, 1 030
// with 8 192 per list, 1 016 so).
static int scan_blocks(int64_t nnz) { return (int)((nnz + 1 + kScanTile - 1) / kScanTile); }

// Long lists: a wave looks at 64 neighbouring positions in each of kLooks places.
constexpr int kLooks = 8;
constexpr int64_t kLookEdges = (int64_t)8192 * kScanTile;
__global__ __launch_bounds__(2 * kLooks * kWave) void k_first_look(const int32_t *in_op, int64_t nnz_in, const int32_t *out_op, int64_t nnz_out, int32_t *status)
{
    __shared__ int32_t s_status[kStatusEnd];
    if (threadIdx.x < kStatusEnd) s_status[threadIdx.x] = 0;
    __syncthreads();
    const int wave = threadIdx.x >> 6, list = wave / kLooks, place = wave % kLooks;
    const int32_t *ops = list ? out_op : in_op;
    const int64_t nnz = list ? nnz_out : nnz_in;
    if (nnz > kLookEdges) {
        const int64_t e = (nnz - 1 - kWave) / (kLooks - 1) * place + lane_id();
        if (ballot64(ops[e] > ops[e + 1]) != 0 && lane_id() == 0) {
            s_status[list ? kStatusOutUnsorted : kStatusInUnsorted] = 1;
            s_status[list ? kStatusLeaveOut : kStatusLeaveIn] = 1;
        }
    }
    __syncthreads();
    if (threadIdx.x < kStatusEnd) status[threadIdx.x] = s_status[threadIdx.x];
}

hipError_t launch_first_look(const EdgeList &in, const EdgeList &out, int32_t *status, hipStream_t s)
{
    const bool looks = in.nnz > kLookEdges || out.nnz > kLookEdges;
    hipLaunchKernelGGL(k_first_look, dim3(1), dim3(looks ? 2 * kLooks * kWave : kStatusEnd), 0, s, in.op, in.nnz, out.op, out.nnz, status);
    return hipGetLastError();
}

hipError_t launch_scan_edges(const EdgeList *in, const EdgeList &out, int32_t *status, hipStream_t s, bool maybe_left)
{
    const int in_blocks = in ? scan_blocks(in->nnz) : 0;
    int out_blocks = scan_blocks(out.nnz);
    if (maybe_left && out_blocks > 8192) out_blocks = 8192;             // (those that find the list left cost 0.2 ns each)
    const dim3 grid((unsigned)(in_blocks + out_blocks));
    const size_t written = (in ? (size_t)in->nnz * 4 : 0) + (size_t)out.nnz * 8 + (size_t)out.num_ops * 8 + (size_t)out.num_tensors * 8;
    if (written > kStreamBytes)
        hipLaunchKernelGGL(k_scan_edges<true>, grid, dim3(kScanThreads), 0, s, in ? *in : out, out, in_blocks, status + kStatusLeaveIn, status);
    else
        hipLaunchKernelGGL(k_scan_edges<false>, grid, dim3(kScanThreads), 0, s, in ? *in : out, out, in_blocks, status + kStatusLeaveIn, status);
    return hipGetLastError();
}

// The outputs in operator order, every operator's tensors ascending: where tensors are numbered as they are created, this
// is the order by tensor, and takes a look at the neighbours where a sort takes three passes over the list.
// What bounds it are the loads: a thread takes four positions and asks for the four on either side of them at once, and
// only an operator whose row is not inside that window has its row walked (25 M outputs, one to three per operator: 196 us
// one entry after the other, now 95).
constexpr int kMaxRow = 64;
constexpr int kOrderThreads = 256;

__global__ __launch_bounds__(kOrderThreads) void k_order_rows(const int32_t *ops, const int32_t *tensors, int64_t nnz,
                                                               int32_t *keys, int32_t *status)
{
    if (status[0] & kErrIdRange) return;                                  // (an operator -1 would be taken for a place beyond the list)
    constexpr int kPer = 4, kSpan = 3 * kPer;
    const bool wide = ((reinterpret_cast<uintptr_t>(ops) | reinterpret_cast<uintptr_t>(tensors)) & 15) == 0;
    const int64_t gsize = (int64_t)gridDim.x * kOrderThreads * kPer;
    bool moved = false, longer = false;
    for (int64_t e0 = ((int64_t)blockIdx.x * kOrderThreads + threadIdx.x) * kPer; e0 < nnz; e0 += gsize) {
        int32_t o[kSpan], t[kSpan];                         // of the positions e0 - 4 ... e0 + 7; -1: none there
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int64_t at = e0 + (q - 1) * kPer;
            if (wide && at >= 0 && at + kPer <= nnz) {
                const int4 a = *reinterpret_cast<const int4 *>(ops + at), b = *reinterpret_cast<const int4 *>(tensors + at);
                o[4 * q] = a.x; o[4 * q + 1] = a.y; o[4 * q + 2] = a.z; o[4 * q + 3] = a.w;
                t[4 * q] = b.x; t[4 * q + 1] = b.y; t[4 * q + 2] = b.z; t[4 * q + 3] = b.w;
            } else {
#pragma unroll
                for (int j = 0; j < kPer; ++j) {
                    const bool there = at + j >= 0 && at + j < nnz;
                    o[4 * q + j] = there ? ops[at + j] : -1;
                    t[4 * q + j] = there ? tensors[at + j] : 0;
                }
            }
        }
#pragma unroll
        for (int j = kPer; j < 2 * kPer; ++j) {
            const int64_t e = e0 + j - kPer;
            if (e >= nnz) continue;
            int before = 0, below = 0;                      // entries of the row before this one; how many sort before it
            if (o[0] == o[j] || o[kSpan - 1] == o[j]) {     // the row may go on beyond the window
                int n = 1;
                for (int64_t i = e - 1; i >= 0 && n <= kMaxRow && ops[i] == o[j]; --i, ++n, ++before) below += tensors[i] <= t[j];
                for (int64_t i = e + 1; i < nnz && n <= kMaxRow && ops[i] == o[j]; ++i, ++n) below += tensors[i] < t[j];
                if (n > kMaxRow) {
                    longer = true;
                    below = before;
                }
            } else {
#pragma unroll
                for (int i = 1; i < kSpan - 1; ++i) {
                    const bool same = o[i] == o[j];
                    before += same && i < j;
                    below += same && (i < j ? t[i] <= t[j] : i > j && t[i] < t[j]);
                }
            }
            moved |= below != before;
            keys[e + (below - before)] = t[j];
        }
    }
    if (ballot64(moved) != 0 && lane_id() == 0 && load_coherent(&status[kStatusScattered]) == 0)
        store_coherent(&status[kStatusScattered], 1);
    if (ballot64(longer) != 0 && lane_id() == 0) store_coherent(&status[kStatusProdUnsorted], 1);
}

hipError_t launch_order_rows(const int32_t *ops, const int32_t *tensors, int64_t nnz, int32_t *keys, int32_t *status, hipStream_t s)
{
    if (nnz == 0) return hipSuccess;
    int64_t blocks = (nnz + kOrderThreads * 4 - 1) / (kOrderThreads * 4);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_order_rows, dim3((unsigned)blocks), dim3(kOrderThreads), 0, s, ops, tensors, nnz, keys, status);
    return hipGetLastError();
}

// Row pointers from keys in row order: rowptr[r] = first position whose key is >= r, rowptr[n_rows] = nnz.
// Position i writes the rows (keys[i-1], keys[i]]; gaps longer than a few rows are filled by the whole wave.
__global__ __launch_bounds__(256) void k_row_bounds(const int32_t *keys, int64_t nnz, int32_t n_rows, int32_t *rowptr, const int32_t *status)
{
    if (status[0] & kErrIdRange) return;                                              // (a key that is no row)
    // a thread takes four neighbouring positions per step (one 16-byte load when the keys are aligned for it): with a
    // single position per thread the pass waits for memory most of its time
    constexpr int kPer = 4;
    const bool wide = (reinterpret_cast<uintptr_t>(keys) & 15) == 0;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x * kPer;
    const int64_t steps = (nnz + 1 + gsize - 1) / gsize;                // position nnz closes the last rows
    for (int64_t st = 0; st < steps; ++st) {                            // whole waves stay in the loop
        const int64_t i0 = st * gsize + ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kPer;
        int32_t k[kPer + 1];                                            // k[j] = key before position i0 + j
        if (i0 <= nnz) k[0] = i0 == 0 ? -1 : keys[i0 - 1];
        if (wide && i0 + kPer <= nnz) {
            const int4 v = *reinterpret_cast<const int4 *>(keys + i0);
            k[1] = v.x; k[2] = v.y; k[3] = v.z; k[4] = v.w;
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) k[j + 1] = i0 + j < nnz ? keys[i0 + j] : n_rows;
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            int lo = 0, hi = -1;                                        // rows lo..hi get the value i0 + j
            if (i0 + j <= nnz) {
                lo = k[j] + 1;
                hi = k[j + 1];
            }
            write_rows(rowptr, lo, hi, (int32_t)(i0 + j));
        }
    }
}

hipError_t launch_row_bounds(const int32_t *keys, int64_t nnz, int32_t n_rows, int32_t *rowptr, const int32_t *status, hipStream_t s)
{
    int64_t blocks = (nnz + 1 + 1023) / 1024;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_row_bounds, dim3((unsigned)blocks), dim3(256), 0, s, keys, nnz, n_rows, rowptr, status);
    return hipGetLastError();
}

// Both ids of every edge of a list that is sorted as a whole.
__global__ __launch_bounds__(256) void k_check_ids(const int32_t *ops, const int32_t *tensors, int64_t nnz, int32_t num_ops,
                                                    int32_t num_tensors, int32_t *status)
{
    bool bad = false;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * 256)
        bad |= (uint32_t)ops[e] >= (uint32_t)num_ops || (uint32_t)tensors[e] >= (uint32_t)num_tensors;
    if (ballot64(bad) != 0 && lane_id() == 0) atomicOr(status, kErrIdRange);
}

hipError_t launch_check_ids(const EdgeList &l, int32_t *status, hipStream_t s)
{
    if (l.nnz == 0) return hipSuccess;
    const int64_t blocks = (l.nnz + 255) / 256;
    hipLaunchKernelGGL(k_check_ids, dim3((unsigned)(blocks < 8192 ? blocks : 8192)), dim3(256), 0, s, l.op, l.tensor, l.nnz, l.num_ops,
                       l.num_tensors, status);
    return hipGetLastError();
}

// Borrowed CSR: rowptr[0] == 0, monotone, rowptr[n_rows] == nnz, every idx in [0, n_vals), and whether the outputs are one run of tensors.
// All four arrays in one launch, a workgroup per 4 096 entries, sixteen bytes per load: the arrays are read once, at the rate of
// memory (50 M operators, 1.3 GB: 450 us with 8 192 workgroups and an entry per load, 283 so; 366 with 1 024 entries per workgroup).
constexpr int kCsrTile = 4 * kScanTile;
struct CsrTiles { int32_t in_idx, out_row, out_idx; };                 // first tiles of the arrays behind in_rowptr
__global__ __launch_bounds__(kScanThreads) void k_check_csr(GraphView g, CsrTiles tiles, int32_t *status)
{
    __shared__ int s_scattered;
    constexpr int kPer = 4, kAtOnce = kCsrTile / kScanTile;
    if (threadIdx.x == 0) s_scattered = 0;
    __syncthreads();
    const int tile = blockIdx.x;
    // (an array without entries has no tile, and begins where the next one does)
    const int which = tile < tiles.in_idx ? 0 : tile < tiles.out_row ? 1 : tile < tiles.out_idx ? 2 : 3;
    const int first = which == 0 ? 0 : which == 1 ? tiles.in_idx : which == 2 ? tiles.out_row : tiles.out_idx;
    const bool in = which < 2, rows = which == 0 || which == 2;
    const int32_t *p = which == 0 ? g.in_rowptr : which == 1 ? g.in_idx : which == 2 ? g.out_rowptr : g.out_idx;
    const int32_t nnz = in ? g.nnz_in : g.nnz_out;
    const int64_t n = rows ? (int64_t)g.num_ops + 1 : nnz;
    int32_t v[kAtOnce][kPer + 1];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
        const int64_t e0 = (int64_t)(tile - first) * kCsrTile + q * kScanTile + threadIdx.x * kPer;
        if (((uintptr_t)p & 15) == 0 && e0 + kPer <= n) {
            const int4 x = *reinterpret_cast<const int4 *>(p + e0);
            v[q][0] = x.x; v[q][1] = x.y; v[q][2] = x.z; v[q][3] = x.w;
        } else {
#pragma unroll
            for (int j = 0; j < kPer; ++j) v[q][j] = e0 + j < n ? p[e0 + j] : 0;
        }
        v[q][kPer] = rows && e0 + kPer < n ? p[e0 + kPer] : 0;
    }
    const int32_t shift = g.num_tensors - g.nnz_out;
    int bad = 0;
    bool scattered = false;
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
        const int64_t e0 = (int64_t)(tile - first) * kCsrTile + q * kScanTile + threadIdx.x * kPer;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int64_t e = e0 + j;
            const int32_t x = v[q][j];
            if (e >= n) break;
            if (rows) {
                if (x < 0 || x > nnz || (e == 0 && x != 0) || (e == n - 1 ? x != nnz : v[q][j + 1] < x)) bad |= kErrCsr;
            } else {
                if (x < 0 || x >= g.num_tensors) bad |= kErrIdRange;
                scattered |= x != (int32_t)e + shift;
            }
        }
    }
    if (bad) atomicOr(status, bad);
    if (rows || in) return;                                             // (the same in every thread)
    if (ballot64(scattered) != 0 && lane_id() == 0) s_scattered = 1;
    __syncthreads();
    if (threadIdx.x < 2 && s_scattered) {
        int32_t *word = status + (threadIdx.x ? kStatusScattered : kStatusNoRun);
        if (load_coherent(word) == 0) store_coherent(word, 1);
    }
}

hipError_t launch_check_csr(const GraphView &g, int32_t *status, hipStream_t s)
{
    auto of = [](int64_t n) { return (int32_t)((n + kCsrTile - 1) / kCsrTile); };
    CsrTiles t{of((int64_t)g.num_ops + 1), 0, 0};
    t.out_row = t.in_idx + of(g.nnz_in);
    t.out_idx = t.out_row + of((int64_t)g.num_ops + 1);
    hipLaunchKernelGGL(k_check_csr, dim3((unsigned)(t.out_idx + of(g.nnz_out))), dim3(kScanThreads), 0, s, g, t, status);
    return hipGetLastError();
}

// row_of[e] = r for every entry e of row r (operator id of every entry of an out CSR), long rows by whole waves (a thread takes
// 0.1 us per entry: 2 000 outputs of one operator 250 us, now 3); -1 everywhere if the CSR is none, or an index of it is
// out of range (status[0]): the pass over this list then reports that again, and touches nothing.
// run_idx, run_row (or NULL): where the outputs are one run of tensors these are the rows by tensor, finished here, and the pass over the
// list is told to leave it (50 M operators, borrowed: 1 050 -> 590 us with what k_check_csr gains).
__global__ __launch_bounds__(256) void k_expand_rows(const int32_t *rowptr, int32_t n_rows, int32_t nnz, int32_t *row_of, int32_t *run_idx,
                                                     int32_t *run_row, int32_t num_tensors, int32_t *status)
{
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x, gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (status[0] & (kErrCsr | kErrIdRange)) {
        for (int64_t e = gtid; e < nnz; e += gsize) row_of[e] = -1;
        return;
    }
    const bool run = run_idx && status[kStatusNoRun] == 0;
    if (run) {
        const int32_t shift = num_tensors - nnz;
        for (int64_t t = gtid * 4; t <= num_tensors; t += gsize * 4) {  // (run_row begins the caller's storage)
            auto row = [&](int64_t at) { return (int32_t)max(at - shift, (int64_t)0); };
            if (t + 4 <= num_tensors) {
                store16<false>(run_row + t, row(t), row(t + 1), row(t + 2), row(t + 3));
            } else {
                for (int64_t at = t; at <= num_tensors; ++at) run_row[at] = row(at);
            }
        }
        if (gtid == 0) status[kStatusLeaveOut] = 1;
        row_of = run_idx;
    }
    for (int64_t r = gtid; r - lane_id() < n_rows; r += gsize) {            // whole waves stay in the loop
        const bool is = r < n_rows;
        write_rows(row_of, is ? rowptr[r] : 0, (is ? rowptr[r + 1] : 0) - 1, (int32_t)r);
    }
}

hipError_t launch_expand_rows(const int32_t *rowptr, int32_t n_rows, int32_t nnz, int32_t *row_of, int32_t *run_idx, int32_t *run_row,
                              int32_t num_tensors, int32_t *status, hipStream_t s)
{
    int64_t blocks = ((int64_t)n_rows + 255) / 256;
    const int64_t tensors = run_row ? ((int64_t)num_tensors / 4 + 256) / 256 : 0;
    if (blocks < tensors) blocks = tensors;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_expand_rows, dim3((unsigned)blocks), dim3(256), 0, s, rowptr, n_rows, nnz, row_of, run_idx, run_row, num_tensors, status);
    return hipGetLastError();
}

// Did the pass over the edges leave finished rows (and producer words)?  What it wrote is not to be trusted otherwise: the
// kernels behind it ask before they use it, so that the host need not wait for the answer in between.
__device__ __forceinline__ bool adjacency_ready(const int32_t *status, bool producers)
{
    int v = status[0] | status[kStatusInUnsorted] | status[kStatusOutUnsorted] | status[kStatusInGap] | status[kStatusOutGap] |
            status[kStatusPending];
    if (producers) v |= status[kStatusProdUnsorted] | status[kStatusProdGap];
    return v == 0;
}

// Topological precondition (Sec. 3.2: operators run in creation order): every producer of an
// operator's input was created before the operator.
__global__ __launch_bounds__(256) void k_check_topological(GraphView g, int32_t *error)
{
    if (!adjacency_ready(error, true)) return;
    g.run_shift = error[kStatusNoRun] == 0 ? g.num_tensors - g.nnz_out : -1;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < g.num_ops; o += gsize) {
        for (int32_t e = g.in_rowptr[o]; e < g.in_rowptr[o + 1]; ++e) {
            const int32_t t = g.in_idx[e];
            if (t < 0 || t >= g.num_tensors) continue;      // reported by the range check
            const int32_t pr = producer_of(g, t);           // one word instead of two CSR hops
            if (pr >= 0) {
                if (pr >= o) bad = true;
            } else if (pr == kMulti) {
                for (int32_t p = g.prod_rowptr[t]; p < g.prod_rowptr[t + 1]; ++p)
                    if (g.prod_idx[p] >= o) bad = true;
            }
        }
    }
    if (bad) atomicOr(error, kErrTopo);
}

hipError_t launch_check_topological(const GraphView &g, int32_t *error, hipStream_t s)
{
    if (g.num_ops == 0) return hipSuccess;
    int64_t blocks = ((int64_t)g.num_ops + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_check_topological, dim3((unsigned)blocks), dim3(256), 0, s, g, error);
    return hipGetLastError();
}

// Packed batch: every edge of an operator of graph g must touch a tensor of graph g.
__device__ __forceinline__ int find_graph(const int64_t *off, int num_graphs, int64_t id)
{
    int lo = 0, hi = num_graphs;          // largest g with off[g] <= id
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= id) lo = mid; else hi = mid;
    }
    return lo;
}

// How far back do operators read?  Sampled (the first input of a few thousand operators, spread over the graph) for the
// traversal's schedule and the choice between it and the sweep.  has: this lane's operator has an input, its first is `t`; o is
// its number among its graph's num_ops operators, whose num_outputs outputs are numbered in creation order from t_first on, own the
// first that it writes.
constexpr int kSoonTensors = 8;
__device__ __forceinline__ void sample_reach(bool has, int64_t o, int32_t t, int64_t num_ops, int32_t t_first, int64_t num_outputs,
                                             int32_t own, int32_t *status)
{
    has = has && t >= t_first;                              // (graph inputs have no producer)
    const float back = (float)o / (float)num_ops - (float)(t - t_first) / (float)num_outputs;
    const u64 seen = ballot64(has);
    auto count = [&](bool is, int word) {
        const u64 m = ballot64(has && is);
        if (lane_id() == 0 && m) atomicAdd(&status[word], __popcll(m));
    };
    if (seen == 0) return;
    if (lane_id() == 0) atomicAdd(&status[kStatusSampled], __popcll(seen));
    count(back < 1.0f / 8, kStatusWithin8);
    count(back < 1.0f / 32, kStatusWithin32);
    count(back < 1.0f / 192, kStatusWithin192);
    count(back < 1.0f / 640, kStatusWithin640);
    count(back < 1.0f / 2048, kStatusWithin2048);
    count(own - t <= kSoonTensors, kStatusSoon);
}
constexpr int kSampleWaves = 32;         // (updates of one address take 11 ns each)

// Neighbouring operators of one place in a single graph whose outputs are one run per wave, the places evenly spread.
__device__ __forceinline__ void sample_single(const GraphView &g, int place, int places, int32_t *status)
{
    const int32_t shift = g.num_tensors - g.nnz_out;
    const int64_t o = (int64_t)((double)g.num_ops * place / places) + lane_id();
    const bool in_range = o < g.num_ops;
    const int32_t ib = in_range ? g.in_rowptr[o] : 0, ie = in_range ? g.in_rowptr[o + 1] : 0;
    sample_reach(ie > ib, o, ie > ib ? g.in_idx[ib] : 0, g.num_ops, shift, g.nnz_out,
                 (in_range ? g.out_rowptr[o] : 0) + shift, status);
}

// ... where there are no records to be made
__global__ __launch_bounds__(kWave) void k_sample_reach(GraphView g, int32_t *status)
{
    if (adjacency_ready(status, false) && status[kStatusScattered] == 0) sample_single(g, blockIdx.x, gridDim.x, status);
}

static int record_blocks(int64_t num_ops) { return (int)(num_ops + 255 < (int64_t)2048 * 256 ? (num_ops + 255) / 256 : 2048); }

// The outputs have turned out not to be one run of tensors: producer words that the pass over them left out, taking it for one.  Where no
// tensor has several producers those are the last ones of the list (a list without gaps from somewhere on); else any whose place says so.
// Where they begin is a chain of reads that every wave waits for: 64 places at a time, 3 reads instead of 18 (200 000 operators, an
// input tensor every 64: the build 53.9 -> 51.9 us; 5 M 189 -> 186).  A whole wave comes here.
__device__ __forceinline__ void fill_spared_words(const GraphView &g, int32_t *prod1, const int32_t *status, int64_t gtid, int64_t gsize)
{
    if (!prod1 || !adjacency_ready(status, true)) return;
    const int32_t shift = g.num_tensors - g.nnz_out;
    int64_t lo = max(0, -shift), hi = g.nnz_out;
    while (status[kStatusMulti] == 0 && hi > lo) {          // first position e whose tensor is e + shift: 64 looks at a time
        const int64_t step = (hi - lo + kWave) / kWave;     // (the last look is at hi or behind it)
        const int64_t at = lo + (lane_id() + 1) * step - 1;
        const int c = __ffsll((unsigned long long)__ballot(at >= hi || g.prod_rowptr[at + shift] == at)) - 1;
        hi = min(hi, lo + (c + 1) * step - 1);
        lo += c * step;
    }
    for (int64_t e = lo + gtid; e < g.nnz_out; e += gsize)
        if (g.prod_rowptr[e + shift] == e && g.prod_rowptr[e + shift + 1] == e + 1) prod1[e + shift] = g.prod_idx[e];
}

hipError_t launch_sample_reach(const GraphView &g, int32_t *status, hipStream_t s)
{
    const int blocks = record_blocks(g.num_ops);
    if (g.num_ops > 0)
        hipLaunchKernelGGL(k_sample_reach, dim3((unsigned)(blocks < kSampleWaves ? blocks : kSampleWaves)), dim3(kWave), 0, s, g, status);
    return hipGetLastError();
}

// Single graphs.  Outputs that are one run of tensors have no records.
template <bool kStream>
__global__ __launch_bounds__(256) void k_build_records(GraphView g, Quad *orec, int32_t *prod1, int32_t *status)
{
    if (!adjacency_ready(status, false)) return;
    if (status[kStatusScattered] == 0 && blockIdx.x < kSampleWaves && threadIdx.x < kWave)
        sample_single(g, blockIdx.x, min((int)gridDim.x, kSampleWaves), status);
    if (status[kStatusNoRun] == 0) return;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x, gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t o = gtid; o < g.num_ops; o += gsize) {
        const int32_t ib = g.in_rowptr[o], ie = g.in_rowptr[o + 1];
        const int32_t ob = g.out_rowptr[o], oe = g.out_rowptr[o + 1];
        const int32_t first = oe > ob ? g.out_idx[ob] : 0;
        bool consecutive = true;
        for (int32_t e = ob + 1; e < oe; ++e) consecutive &= g.out_idx[e] == first + (e - ob);
        write_record<kStream>(&orec[o], ib, ie, ob, oe, first, consecutive);
    }
    fill_spared_words(g, prod1, status, gtid, gsize);
}

hipError_t launch_build_records(const GraphView &g, Quad *orec, int32_t *prod1, int32_t *status, hipStream_t s)
{
    if (g.num_ops == 0) return hipSuccess;
    const int blocks = record_blocks(g.num_ops);
    if ((size_t)g.num_ops * sizeof(int4) > kStreamBytes)
        hipLaunchKernelGGL(k_build_records<true>, dim3((unsigned)blocks), dim3(256), 0, s, g, orec, prod1, status);
    else
        hipLaunchKernelGGL(k_build_records<false>, dim3((unsigned)blocks), dim3(256), 0, s, g, orec, prod1, status);
    return hipGetLastError();
}

// Producer words from the tensors' rows (where the pass over the edges did not write them)
__global__ __launch_bounds__(256) void k_build_producers(GraphView g, int32_t *prod1, int32_t *status)
{
    if (status[0] & kErrIdRange) return;                    // (no rows: whatever the memory held before)
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < g.num_tensors; t += gsize) {
        const int32_t pb = g.prod_rowptr[t], pe = g.prod_rowptr[t + 1];
        int32_t r = kNoProducer;
        if (pe - pb == 1) {
            r = g.prod_idx[pb];
        } else if (pe - pb > 1) {
            r = kMulti;
            status[kStatusMulti] = 1;                       // (the same value from every writer)
        }
        prod1[t] = r;
    }
}

hipError_t launch_build_producers(const GraphView &g, int32_t *prod1, int32_t *status, hipStream_t s)
{
    if (g.num_tensors == 0) return hipSuccess;
    int64_t blocks = ((int64_t)g.num_tensors + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_build_producers, dim3((unsigned)blocks), dim3(256), 0, s, g, prod1, status);
    return hipGetLastError();
}

// Records (unless the outputs are one run) of a packed batch, or of a single graph that the ring sweep may take, and in the same walk over the edges: does
// every edge of an operator of graph g touch a tensor of graph g, and whether and how the ring sweep can take the graphs
// (status words from kStatusRing on; see ring_sweep.hip): are the outputs of every graph one run of tensors that ends
// with its last one, how many tensors lie before that run, how far below the end of its own outputs does an operator read,
// and how many outputs do 64 neighbouring operators have.  Outputs in one run of which no operator reads its own or a
// later one are a topological order, which spares a batch the look at every input's producer.
// The reading of the adjacency bounds it on a large batch (100 000 operators of small graphs: launch and latency).  Workgroups report once each: a look at the status words
// by every wave was a quarter of the build of a middling batch (27 000 waves: 80 us).
constexpr int kCheckThreads = 256;

template <bool kStream>
__global__ __launch_bounds__(kCheckThreads) void k_records_and_check(GraphView g, Quad *orec, int32_t *ofirst, int32_t *prod1, int32_t *status)
{
    __shared__ int s_found[6];                      // error, scattered, low, dist, span64, reach
    if (!adjacency_ready(status, false)) return;
    const bool records = status[kStatusNoRun] != 0;
    if (threadIdx.x < 6) s_found[threadIdx.x] = 0;
    __syncthreads();
    // a wave walks a contiguous stretch of operators 64 at a time, so a lane's graph index only ever steps
    // forward: one binary search per lane, not one per operator
    const bool batched = g.num_graphs > 1;
    const int64_t waves = (int64_t)gridDim.x * (kCheckThreads / kWave);
    const int64_t wave_id = (int64_t)blockIdx.x * (kCheckThreads / kWave) + (threadIdx.x >> 6);
    const int64_t per = (((int64_t)g.num_ops + waves - 1) / waves + kWave - 1) / kWave * kWave;
    const int64_t begin = wave_id * per, last = min(begin + per, (int64_t)g.num_ops);
    bool bad = false, scattered = false;
    int low = 0, dist = 0, span64 = 0, reach = 0;
    int gi = 0;
    int64_t lo = 0, hi = g.num_tensors, o_lo = 0, o_hi = g.num_ops;
    int32_t shift = 0, t_first = 0;                         // output edge e should be tensor e + shift
    auto enter = [&](int64_t o) {                           // the graph of o, gi or one behind it
        if (batched) {
            while (o >= g.op_off[gi + 1]) ++gi;             // op_off[num_graphs] == num_ops > o: stops in range
            lo = g.t_off[gi];
            hi = g.t_off[gi + 1];
            o_lo = g.op_off[gi];
            o_hi = g.op_off[gi + 1];
        }
        shift = (int32_t)hi - g.out_rowptr[o_hi];
        t_first = g.out_rowptr[o_lo] + shift;
        if (t_first < lo) scattered = true;                 // more outputs than tensors
        low = max(low, t_first - (int32_t)lo);
    };
    // (at the first operators of some of the waves; a batch of 64 graphs and more goes one way whatever it reads)
    const bool samples = (batched ? g.num_graphs < 64 : status[kStatusScattered] == 0) &&
                         wave_id % ((waves + kSampleWaves - 1) / kSampleWaves) == 0;
    // A wave's time was that of its memory accesses, two and three after each other for every 64 operators: rows are asked for two
    // steps ahead, the first entries of rows one step ahead (82 M operators: 1.00 -> 0.75 ms = 4.2 TB/s).
    struct Row { int32_t ib, ie, ob, oe; };
    struct Entries { int32_t t[4], u[2]; };
    // (the row behind the last operator begins where the lists end: a stretch of 64 operators may end there)
    auto row_of = [&](int64_t o) {
        Row r{g.nnz_in, g.nnz_in, g.nnz_out, g.nnz_out};
        if (o < g.num_ops) r = Row{g.in_rowptr[o], g.in_rowptr[o + 1], g.out_rowptr[o], g.out_rowptr[o + 1]};
        return r;
    };
    // (an operator without inputs or outputs looks at a neighbour's entry and does not use it)
    const int32_t none_in = max(g.nnz_in - 1, 0), none_out = max(g.nnz_out - 1, 0);
    auto entries_of = [&](const Row &r) {
        Entries x{};
        if (g.nnz_in > 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) x.t[j] = g.in_idx[min(r.ib + j, none_in)];
        }
        if (g.nnz_out > 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) x.u[j] = g.out_idx[min(r.ob + j, none_out)];
        }
        return x;
    };
    Row next{}, after{};
    Entries next_entries{};
    if (begin < last) {                                     // wave-uniform, as the two below
        next = row_of(begin + lane_id());
        if (begin + kWave < last) after = row_of(begin + kWave + lane_id());
        const int64_t o = min(begin + lane_id(), last - 1);
        if (batched) gi = find_graph(g.op_off, g.num_graphs, o);
        enter(o);                                           // (asked for before the wait for the rows)
        next_entries = entries_of(next);
    }
    for (int64_t base = begin; base < last; base += kWave) {
        const int64_t o = base + lane_id();
        const int32_t ib = next.ib, ie = next.ie, ob = next.ob, oe = next.oe;
        const Entries x = next_entries;
        const int32_t *t = x.t, *u = x.u;
        if (base + kWave < last) {
            next = after;
            next_entries = entries_of(next);
            if (base + 2 * kWave < last) after = row_of(o + 2 * kWave);
        }
        if (o >= last) break;                               // (the last step)
        if (o >= o_hi) enter(o);
        if (samples && o - lane_id() == begin)
            sample_reach(ie > ib, o - o_lo, t[0], o_hi - o_lo, t_first, hi - t_first, ob + shift, status);
        auto input = [&](int32_t x) {
            if (x < lo || x >= hi) bad = true;
            if (x >= t_first) {
                if (x >= ob + shift) scattered = true;      // not written before, if the outputs are one run
                dist = max(dist, oe + shift - x);
                reach = max(reach, ob + shift - x);
            }
        };
        bool consecutive = true;
        const int32_t first = oe > ob ? u[0] : 0;
        auto output = [&](int32_t e, int32_t y) {
            if (y < lo || y >= hi) bad = true;
            if (y != e + shift) scattered = true;
            consecutive &= y == first + (e - ob);
        };
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (ib + j < ie) input(t[j]);
        for (int32_t e = ib + 4; e < ie; ++e) input(g.in_idx[e]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (ob + j < oe) output(ob + j, u[j]);
        for (int32_t e = ob + 2; e < oe; ++e) output(e, g.out_idx[e]);
        if (records && orec) write_record<kStream>(&orec[o], ib, ie, ob, oe, first, consecutive);
        else if (records) ofirst[o] = consecutive ? first : -1;
        if (((o - o_lo) & (kWave - 1)) == 0)                // (the outputs of 64 operators end where those of the next begin)
            span64 = max(span64, (o + kWave <= o_hi && base + kWave < last ? next.ob : g.out_rowptr[min(o + kWave, o_hi)]) - ob);
    }
    if (records) fill_spared_words(g, prod1, status, (int64_t)blockIdx.x * kCheckThreads + threadIdx.x, (int64_t)gridDim.x * kCheckThreads);
    const int wlow = wave_max(low), wdist = wave_max(dist), wspan = wave_max(span64), wreach = wave_max(reach);
    const bool wbad = ballot64(bad) != 0, wscattered = ballot64(scattered) != 0;
    if (lane_id() == 0) {
        if (wbad) s_found[0] = 1;
        if (wscattered) s_found[1] = 1;
        atomicMax(&s_found[2], wlow);
        atomicMax(&s_found[3], wdist);
        atomicMax(&s_found[4], wspan);
        atomicMax(&s_found[5], wreach);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_found[0]) atomicOr(&status[0], kErrCrossGraph);
    if (threadIdx.x < 5) {                                  // one look, and an atomic only where it would change something
        const int v = s_found[1 + threadIdx.x], at = threadIdx.x < 4 ? kStatusRing + (int)threadIdx.x : (int)kStatusReach;
        if (v > load_coherent(&status[at])) atomicMax(&status[at], v);
    }
}

hipError_t launch_records_and_check(const GraphView &g, Quad *orec, int32_t *ofirst, int32_t *prod1, int32_t *status, int num_cus, hipStream_t s)
{
    if (g.num_ops == 0) return hipSuccess;
    int64_t blocks = ((int64_t)g.num_ops + kCheckThreads - 1) / kCheckThreads;
    if (blocks > 8 * num_cus) blocks = 8 * num_cus;
    if ((size_t)g.num_ops * sizeof(int4) > kStreamBytes)
        hipLaunchKernelGGL(k_records_and_check<true>, dim3((unsigned)blocks), dim3(kCheckThreads), 0, s, g, orec, ofirst, prod1, status);
    else
        hipLaunchKernelGGL(k_records_and_check<false>, dim3((unsigned)blocks), dim3(kCheckThreads), 0, s, g, orec, ofirst, prod1, status);
    return hipGetLastError();
}

}  // namespace dgn
