// What a graph runtime reads off a prune result (Sec. 3.2 of the paper): the tensors to rename
// "ignore" (written by a surviving operator, used by nothing the targets need) and, per target set,
// the surviving operators in creation order.  Both work on the compacted kept list, so their cost
// follows the pruned graph, not the recorded one (apart from clearing the ignore mask).
#include "common.h"

namespace dgn {

constexpr int kPpThreads = 256;

// ignore[y] |= K[o] & ~M[y] for every output y of every kept operator o; tensors with a new non-zero
// mask are counted (a tensor with several producers is counted once: by the add that found it zero).
// several_producers: some tensor of the graph has; in all other graphs nobody else writes y, and a plain store will do.
// What bounds it is the clearing of the whole mask beforehand.  The walk over the list was twice as long as that while
// every wave added its finds to the one counter (11 ns each; 456 000 operators: 173 us -> 67, a workgroup each).
constexpr int kIgThreads = 1024;

__global__ __launch_bounds__(kIgThreads) void k_ignore_mask(GraphView g, bool several_producers, const int32_t *kept_ops,
                                                            const u64 *kept_masks, const int64_t *kept_count, const u64 *M,
                                                            u64 *ignore, int64_t *ignore_count)
{
    __shared__ int s_found;
    const int64_t n = *kept_count;
    const int64_t gsize = (int64_t)gridDim.x * kIgThreads;
    if ((int64_t)blockIdx.x * kIgThreads >= n) return;
    if (threadIdx.x == 0) s_found = 0;
    __syncthreads();
    int found = 0;
    for (int64_t i = (int64_t)blockIdx.x * kIgThreads + threadIdx.x; i < n; i += gsize) {
        const int4 r = op_record(g, kept_ops[i]);
        const u64 k = kept_masks[i];
        const int n_out = r.w >= 0 ? r.w : -r.w;
        for (int j = 0; j < n_out; j += 2) {                // the masks of two outputs are fetched together
            const int j1 = min(j + 1, n_out - 1);
            const int32_t y0 = r.w >= 0 ? r.z + j : g.out_idx[r.z + j], y1 = r.w >= 0 ? r.z + j1 : g.out_idx[r.z + j1];
            const u64 i0 = k & ~M[y0], i1 = j1 > j ? k & ~M[y1] : 0;
            if (several_producers) {
                if (i0) found += atomicOr(&ignore[y0], i0) == 0;
                if (i1) found += atomicOr(&ignore[y1], i1) == 0;
            } else {
                if (i0) ignore[y0] = i0;
                if (i1) ignore[y1] = i1;
                found += (i0 != 0) + (i1 != 0);
            }
        }
    }
    const int wfound = wave_sum(found);
    if (wfound && lane_id() == 0) atomicAdd(&s_found, wfound);
    __syncthreads();
    if (threadIdx.x == 0 && s_found && ignore_count) atomicAdd((u64 *)ignore_count, (u64)s_found);
}

// Per-set lists.  The kept list is cut into tiles of 64 entries; a 64x64 bit-matrix transpose gives
// lane q the entries of the tile that belong to set q.  Counts go into a set-major table
// (table[q * tiles + tile]), so that ONE exclusive scan over the table yields, for every set and tile,
// the first slot of that tile's entries in the set's list -- lists laid out set after set.
__global__ __launch_bounds__(kPpThreads) void k_set_count(const u64 *kept_masks, int64_t n, int64_t tiles, int32_t *table)
{
    const int lane = lane_id();
    const int64_t wave_id = (int64_t)blockIdx.x * (kPpThreads / kWave) + (threadIdx.x >> 6);
    const int64_t num_waves = (int64_t)gridDim.x * (kPpThreads / kWave);
    for (int64_t tile = wave_id; tile < tiles; tile += num_waves) {
        const int64_t i = tile * kWave + lane;
        const u64 k = i < n ? kept_masks[i] : 0;
        table[(int64_t)lane * tiles + tile] = __popcll(wave_transpose64(k));
    }
}

// The entries of a tile that belong to one set go out together, from neighbouring lanes into neighbouring slots of the
// set's list.  (A lane per set, each writing its own list entry after entry, sent 64 lanes of a store to 64 cache lines:
// 11 M entries in 64 us, now 34.)  The first workgroup leaves the lists' row pointers; entry 64 * tiles of the table holds the
// total (a launch of their own was 2 to 4 us of the 107 that in-place names, ignore mask and lists of a small graph take).
__global__ __launch_bounds__(kPpThreads) void k_set_scatter(const int32_t *kept_ops, const u64 *kept_masks, int64_t n,
                                                             int64_t tiles, const int32_t *table, int32_t *set_ops,
                                                             int64_t capacity, int64_t *set_rowptr)
{
    const int lane = lane_id();
    if (blockIdx.x == 0 && threadIdx.x <= kWave) set_rowptr[threadIdx.x] = table[(int64_t)threadIdx.x * tiles];
    const int64_t wave_id = (int64_t)blockIdx.x * (kPpThreads / kWave) + (threadIdx.x >> 6);
    const int64_t num_waves = (int64_t)gridDim.x * (kPpThreads / kWave);
    for (int64_t tile = wave_id; tile < tiles; tile += num_waves) {
        const int64_t i = tile * kWave + lane;
        const u64 k = i < n ? kept_masks[i] : 0;
        const int32_t op = i < n ? kept_ops[i] : -1;
        const int first = table[(int64_t)lane * tiles + tile];             // lane q: first slot of the tile's entries of set q
        u64 sets = wave_or(k);
        while (sets) {                                      // wave-uniform; ascending lanes: the list stays in creation order
            const int q = __builtin_ctzll(sets);
            sets &= sets - 1;
            const bool in = (k >> q) & 1;
            const int pos = __builtin_amdgcn_readlane(first, q) + __popcll(ballot64(in) & lanemask_lt());
            if (in && pos < capacity) set_ops[pos] = op;
        }
    }
}

size_t set_lists_scratch_bytes(int64_t num_kept)
{
    const int64_t tiles = (num_kept + kWave - 1) / kWave;
    const size_t table = ((size_t)(64 * tiles + 1) * 4 + 255) & ~(size_t)255;
    return table + scan_tmp_bytes(64 * tiles) + 256;
}

hipError_t launch_ignore_mask(const GraphView &g, bool several_producers, const int32_t *kept_ops, const u64 *kept_masks, const int64_t *kept_count,
                              const u64 *M, u64 *ignore, int64_t *ignore_count, int grid_blocks, hipStream_t s)
{
    FillRegion clr[2] = {{ignore, (size_t)g.num_tensors * 8}, {ignore_count, ignore_count ? sizeof(int64_t) : 0}};
    hipError_t e = launch_clear(clr, 2, s);
    if (e != hipSuccess) return e;
    if (g.num_ops > 0)
        hipLaunchKernelGGL(k_ignore_mask, dim3((unsigned)grid_blocks), dim3(kIgThreads), 0, s, g, several_producers, kept_ops,
                           kept_masks, kept_count, M, ignore, ignore_count);
    return hipGetLastError();
}

hipError_t launch_set_lists(const int32_t *kept_ops, const u64 *kept_masks, int64_t num_kept, int64_t *set_rowptr,
                            int32_t *set_ops, int64_t capacity, void *scratch, int grid_blocks, hipStream_t s)
{
    const int64_t tiles = (num_kept + kWave - 1) / kWave;
    int32_t *table = static_cast<int32_t *>(scratch);
    void *scan_tmp = static_cast<char *>(scratch) + (((size_t)(64 * tiles + 1) * 4 + 255) & ~(size_t)255);
    if (tiles > 0) {
        int64_t blocks = (tiles + (kPpThreads / kWave) - 1) / (kPpThreads / kWave);
        if (blocks > grid_blocks) blocks = grid_blocks;
        hipLaunchKernelGGL(k_set_count, dim3((unsigned)blocks), dim3(kPpThreads), 0, s, kept_masks, num_kept, tiles, table);
        hipError_t e = launch_exclusive_scan(table, table, 64 * tiles, scan_tmp, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_set_scatter, dim3((unsigned)blocks), dim3(kPpThreads), 0, s, kept_ops, kept_masks, num_kept,
                           tiles, table, set_ops, capacity, set_rowptr);
        return hipGetLastError();
    }
    FillRegion none[1] = {{set_rowptr, (kWave + 1) * sizeof(int64_t)}};
    return launch_clear(none, 1, s);
}

}  // namespace dgn
