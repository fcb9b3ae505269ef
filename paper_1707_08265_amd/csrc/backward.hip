// Backward Prune (Sec. 2.3, Algorithm 2 of the paper): for every pair (x_obj, x_wrt) the nodes on a
// route from x_obj to x_wrt are marked; everything else can be eliminated.
//
// A node is on such a route iff x_obj reaches it and it reaches x_wrt.  The second half is what the
// forward prune computes when x_wrt is the only target of set i (its coloured set: everything x_wrt
// depends on), so pair i owns bit i and the first stage is one ordinary 64-set prune with targets
// x_wrt.  The second stage runs forwards from x_obj, but only *inside* that coloured set: every node
// between x_obj and a marked node reaches x_wrt as well, and every operator between two such nodes was
// kept by the first stage.  So the forward stage never leaves the (usually small) kept operator list
// of the first stage and needs no tensor -> consumer adjacency:
//     for every kept operator o:   F[y] |= (OR_{x in in(o)} F[x]) & B[y]    for y in out(o)
// repeated over the list, which is in creation order, until nothing changes.  F is the marked set.
//
// The passes run on the kept operators' numbers in the list, not on tensors.  With FO[i] = the marks that arrive at the
// inputs of the i-th kept operator, cut to its K of the first stage, F[y] = FO[i] & B[y] for its outputs y, and
//     FO[i] = K[i] & (seeds at its inputs | OR of FO over the producers of its inputs):
// the cut with B at a tensor between two operators may be left out, because K of the reading operator is a part of it
// already.  So a pass reads one list of operator numbers from end to end and FO, a few MB (a mark of a tensor is one
// cache line in an array as large as the graph), each FO is written by one lane, without atomics, and B and F are
// touched once, when the passes are over.  456 000 kept operators with 1.5 M inputs of a 50 M-operator graph: 17 passes of
// 60 us before, 8 of 36 now (48 us to make the list, 27 to write the marks); the whole call 1.79 ms -> 0.91.
#include "common.h"

namespace dgn {

// rowptr[i] = i, i = 0..n: target set i holds exactly entry i
__global__ __launch_bounds__(64) void k_iota(int32_t *rowptr, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n) rowptr[i] = i;
}

constexpr int kFwThreads = 256;
constexpr int kLinkThreads = 1024;
constexpr int kLinkWaves = kLinkThreads / kWave;

// The kept list's numbers: op_of[o] = 1 + the place of operator o in the list, in the array that held K of the first stage
// (zero for all others); K by place.  The first wave also clears the flags (flags[0]: error bits) and sets the seeds: pair i
// seeds bit i at x_obj when x_obj leads to x_wrt (bit i of B) and the two differ (only children are ever compared with
// x_wrt: a node is not a route to itself).
__global__ __launch_bounds__(kFwThreads) void k_number_kept(const int32_t *kept, const int64_t *kept_count, u64 *place, u64 *Kc,
                                                            int64_t T, int num_pairs, const int32_t *obj, const int32_t *wrt,
                                                            const u64 *B, u64 *F, int32_t *flags)
{
    if (blockIdx.x == 0 && threadIdx.x < kWave) {
        const int i = threadIdx.x;
        const int32_t a = i < num_pairs ? obj[i] : 0, b = i < num_pairs ? wrt[i] : 0;
        const bool bad = i < num_pairs && (a < 0 || a >= T || b < 0 || b >= T);
        const u64 any_bad = ballot64(bad);
        flags[i] = i == 0 && any_bad ? kErrIdRange : 0;
        const u64 bit = (u64)1 << i;
        if (i < num_pairs && !bad && a != b && (B[a] & bit)) atomicOr(&F[a], bit);
    }
    const int64_t n = *kept_count;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsize) {
        const int32_t o = kept[i];
        Kc[i] = place[o];
        place[o] = (u64)(i + 1);
    }
}

// For every group of 64 kept operators the places of the producers of its inputs (one entry per input, with the lane that
// it belongs to), and FO as the seeds alone make it.  An input without a kept producer: -1; with several producers: -2 - its
// id, looked up in every pass.  Groups are one after the other in the list in no particular order: a workgroup reserves
// room for its sixteen groups at once.
__global__ __launch_bounds__(kLinkThreads) void k_link_kept(GraphView g, const int32_t *kept, const int64_t *kept_count,
                                                            const u64 *place, const u64 *F, const int32_t *obj, int num_pairs,
                                                            BackwardLinks b, int32_t *cursor)
{
    __shared__ uint32_t s_seed[64];                 // which tensors may hold a seed: a bit per id modulo 2048
    __shared__ int s_mark[kLinkWaves][kWave];
    __shared__ u64 s_acc[kLinkWaves][kWave];
    __shared__ int s_total[kLinkWaves], s_base;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const int64_t n = *kept_count;
    if (threadIdx.x < 64) s_seed[threadIdx.x] = 0;
    __syncthreads();
    if ((int)threadIdx.x < num_pairs) atomicOr(&s_seed[(obj[threadIdx.x] >> 5) & 63], 1u << (obj[threadIdx.x] & 31));
    for (int64_t base = (int64_t)blockIdx.x * kLinkThreads; base < n; base += (int64_t)gridDim.x * kLinkThreads) {
        const int64_t i = base + threadIdx.x;                           // whole workgroups stay in the loop
        int eb = 0, deg = 0;
        if (i < n) {
            const int4 r = op_record(g, kept[i]);
            eb = r.x;
            deg = r.y;
        }
        const int incl = wave_incl_scan(deg), excl = incl - deg;
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
        s_acc[wave][lane] = 0;
        if (lane == 0) s_total[wave] = total;
        __syncthreads();
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < kLinkWaves; ++w) {
            if (w < wave) before += s_total[w];
            all += s_total[w];
        }
        if (threadIdx.x == 0) s_base = atomicAdd(cursor, all);
        __syncthreads();
        const int start = s_base + before;
        for (int w0 = 0; w0 < total; w0 += kWave) {                     // wave-uniform
            s_mark[wave][lane] = 0;
            __builtin_amdgcn_wave_barrier();
            if (deg > 0 && incl > w0 && excl < w0 + kWave) s_mark[wave][max(excl - w0, 0)] = lane + 1;
            __builtin_amdgcn_wave_barrier();
            const int owner = max(wave_incl_max(s_mark[wave][lane]) - 1, 0);
            __builtin_amdgcn_wave_barrier();
            const int o_eb = __shfl(eb, owner, kWave), o_excl = __shfl(excl, owner, kWave);
            const int e = w0 + lane;
            if (e < total) {
                const int32_t x = g.in_idx[o_eb + (e - o_excl)];
                const int32_t p = producer_of(g, x);
                int32_t link = -1;
                if (p >= 0) link = (int32_t)place[p] - 1;
                else if (p == kMulti) link = -2 - x;
                if ((s_seed[(x >> 5) & 63] >> (x & 31)) & 1) {
                    const u64 f = F[x];
                    if (f) atomicOr(&s_acc[wave][owner], f);
                }
                b.link[start + e] = link;
                b.owner[start + e] = (uint8_t)owner;
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (i < n) b.FO[i] = s_acc[wave][lane] & b.K[i];
        if (lane == 0 && i < n) b.group[i >> 6] = make_int2(start, total);
        __syncthreads();                                                // s_total and s_base are free again
    }
}

// One pass: a wave per group of 64 kept operators, a lane per input entry, the marks gathered per operator in LDS.  Values
// of FO read here may be stale: FO only grows, and the host repeats the pass until one of them changes nothing.  All
// groups of an ordinary kept list are in flight at once, so a pass is a chain of dependent accesses; a wave therefore
// looks again as long as it finds something new, and kFwSweeps times at least (its entries stay in registers, up to
// 64 kFwHeld of them), which lets marks travel several operators within one pass.
constexpr int kFwHeld = 4;
constexpr int kFwSweeps = 3;

__device__ __forceinline__ u64 marks_of(const GraphView &g, int32_t link, const u64 *place, const u64 *FO)
{
    if (link >= 0) return load_coherent(&FO[link]);
    u64 f = 0;
    if (link <= -2) {                                       // several producers
        const int32_t x = -2 - link;
        for (int32_t p = g.prod_rowptr[x]; p < g.prod_rowptr[x + 1]; ++p) {
            const int64_t at = (int64_t)place[g.prod_idx[p]] - 1;
            if (at >= 0) f |= load_coherent(&FO[at]);
        }
    }
    return f;
}

__global__ __launch_bounds__(kFwThreads) void k_forward_pass(GraphView g, const int64_t *kept_count, const u64 *place,
                                                              BackwardLinks b, int32_t *changed)
{
    __shared__ u64 s_acc[kFwThreads / kWave][kWave];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    u64 *acc = s_acc[wave];
    const int64_t n = *kept_count, groups = (n + kWave - 1) >> 6;
    bool added = false;
    for (int64_t gi = (int64_t)blockIdx.x * (kFwThreads / kWave) + wave; gi < groups;
         gi += (int64_t)gridDim.x * (kFwThreads / kWave)) {
        const int2 gr = b.group[gi];
        const int start = gr.x, total = gr.y;
        const int64_t i = gi * kWave + lane;
        const u64 K = i < n ? b.K[i] : 0;
        u64 fo = i < n ? load_coherent(&b.FO[i]) : 0;
        int32_t link[kFwHeld];
        int owner[kFwHeld];
#pragma unroll
        for (int r = 0; r < kFwHeld; ++r) {
            const bool has = r * kWave + lane < total;
            link[r] = has ? b.link[start + r * kWave + lane] : -1;
            owner[r] = has ? b.owner[start + r * kWave + lane] : 0;
        }
        for (int iter = 0; iter < kWave; ++iter) {
            if (ballot64(fo != K) == 0) break;              // nothing can be added any more
            acc[lane] = 0;
            __builtin_amdgcn_wave_barrier();
            u64 f[kFwHeld];
#pragma unroll
            for (int r = 0; r < kFwHeld; ++r) f[r] = marks_of(g, link[r], place, b.FO);
#pragma unroll
            for (int r = 0; r < kFwHeld; ++r)
                if (f[r]) atomicOr(&acc[owner[r]], f[r]);
            for (int e = kFwHeld * kWave + lane; e < total; e += kWave) {
                const u64 more = marks_of(g, b.link[start + e], place, b.FO);
                if (more) atomicOr(&acc[b.owner[start + e]], more);
            }
            __builtin_amdgcn_wave_barrier();
            const u64 nb = acc[lane] & K & ~fo;
            __builtin_amdgcn_wave_barrier();
            if (nb) {
                fo |= nb;
                store_coherent(&b.FO[i], fo);
            }
            const bool any_new = ballot64(nb != 0) != 0;
            added |= any_new;
            if (!any_new && iter + 1 >= kFwSweeps) break;
        }
    }
    if (added && lane == 0) *changed = 1;                   // same value from every writer
}

// The marked masks and K of the result: F[y] |= FO & B[y] for the outputs of every kept operator, K[o] = OR of F over them
// (only where no tensor has several producers: else k_keep_from_list follows); flags as in k_keep_from_list.
__global__ __launch_bounds__(kFwThreads) void k_write_marks(GraphView g, bool several_producers, const int32_t *kept,
                                                            const int64_t *kept_count, const u64 *FO, const u64 *B, u64 *F,
                                                            u64 *K, uint8_t *flags)
{
    const int64_t n = *kept_count;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsize) {
        const int32_t o = kept[i];
        const int4 r = op_record(g, o);
        const u64 fo = FO[i];
        const int n_out = r.w >= 0 ? r.w : -r.w;
        u64 k = 0;
        for (int j = 0; j < n_out; j += 2) {                // the masks of two outputs are fetched together
            const int j1 = min(j + 1, n_out - 1);
            const int32_t y0 = r.w >= 0 ? r.z + j : g.out_idx[r.z + j], y1 = r.w >= 0 ? r.z + j1 : g.out_idx[r.z + j1];
            const u64 a0 = fo & B[y0], a1 = fo & B[y1], f0 = F[y0], f1 = F[y1];
            if (several_producers) {
                if (a0) atomicOr(&F[y0], a0);
                if (a1) atomicOr(&F[y1], a1);
            } else {
                if (a0 & ~f0) F[y0] = f0 | a0;
                if ((a1 & ~f1) && j1 > j) F[y1] = f1 | a1;
                k |= f0 | a0 | f1 | a1;
            }
        }
        if (!several_producers) {
            K[o] = k;
            if (flags && k == 0) flags[o] = 0;
        }
    }
}

// K[o] = OR of F over the outputs of o (removal rule of Sec. 2.1), for the operators of a kept list only; flags
// (or NULL): a byte per operator that is 1 exactly for the operators of the list on entry, 1 where K != 0 on return
__global__ __launch_bounds__(kFwThreads) void k_keep_from_list(GraphView g, const int32_t *kept, const int64_t *kept_count,
                                                                const u64 *F, u64 *K, uint8_t *flags)
{
    const int64_t n = *kept_count;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gsize) {
        const int32_t o = kept[i];
        u64 k = 0;
        for (int32_t e = g.out_rowptr[o]; e < g.out_rowptr[o + 1]; ++e) k |= F[g.out_idx[e]];
        K[o] = k;
        if (flags && k == 0) flags[o] = 0;
    }
}

hipError_t launch_keep_from_list(const GraphView &g, const int32_t *kept, const int64_t *kept_count, const u64 *F, u64 *K,
                                 uint8_t *flags, int grid_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_keep_from_list, dim3((unsigned)grid_blocks), dim3(kFwThreads), 0, s, g, kept, kept_count, F, K,
                       flags);
    return hipGetLastError();
}

hipError_t launch_pair_rows(int num_pairs, int32_t *tgt_rowptr, hipStream_t s)
{
    hipLaunchKernelGGL(k_iota, dim3(2), dim3(64), 0, s, tgt_rowptr, num_pairs);
    return hipGetLastError();
}

BackwardLinks backward_links(void *mem, int64_t P, int64_t Ein, size_t *bytes)
{
    char *p = static_cast<char *>(mem);
    auto take = [&](size_t n) {
        char *r = p;
        p += (n + 255) & ~(size_t)255;
        return r;
    };
    BackwardLinks b;
    b.K = reinterpret_cast<u64 *>(take((size_t)P * 8));
    b.FO = reinterpret_cast<u64 *>(take((size_t)P * 8));
    b.group = reinterpret_cast<int2 *>(take((size_t)(P / kWave + 1) * sizeof(int2)));
    b.link = reinterpret_cast<int32_t *>(take((size_t)Ein * 4));
    b.owner = reinterpret_cast<uint8_t *>(take((size_t)Ein));
    *bytes = (size_t)(p - static_cast<char *>(mem));
    return b;
}

hipError_t launch_link_kept(const GraphView &g, const int32_t *kept, const int64_t *kept_count, u64 *place, const u64 *B, u64 *F,
                            const int32_t *obj, const int32_t *wrt, int num_pairs, const BackwardLinks &b, int32_t *flags,
                            int num_cus, hipStream_t s)
{
    const int64_t most = ((int64_t)g.num_ops + kFwThreads - 1) / kFwThreads, grid = num_cus * 8;
    hipLaunchKernelGGL(k_number_kept, dim3((unsigned)(most < 1 ? 1 : most < grid ? most : grid)), dim3(kFwThreads), 0, s, kept,
                       kept_count, place, b.K, (int64_t)g.num_tensors, num_pairs, obj, wrt, B, F, flags);
    if (g.num_ops == 0) return hipGetLastError();
    const int64_t blocks = ((int64_t)g.num_ops + kLinkThreads - 1) / kLinkThreads;
    hipLaunchKernelGGL(k_link_kept, dim3((unsigned)(blocks < num_cus * 2 ? blocks : num_cus * 2)), dim3(kLinkThreads), 0, s, g,
                       kept, kept_count, place, F, obj, num_pairs, b, flags + 1);
    return hipGetLastError();
}

hipError_t launch_forward_pass(const GraphView &g, const int64_t *kept_count, const u64 *place, const BackwardLinks &b,
                               int32_t *changed, int num_cus, hipStream_t s)
{
    const int64_t most = ((int64_t)g.num_ops + kFwThreads - 1) / kFwThreads, grid = num_cus * 8;
    if (most == 0) return hipSuccess;
    hipLaunchKernelGGL(k_forward_pass, dim3((unsigned)(most < grid ? most : grid)), dim3(kFwThreads), 0, s, g, kept_count, place,
                       b, changed);
    return hipGetLastError();
}

hipError_t launch_write_marks(const GraphView &g, bool several_producers, const int32_t *kept, const int64_t *kept_count,
                              const u64 *FO, const u64 *B, u64 *F, u64 *K, uint8_t *flags, int grid_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_write_marks, dim3((unsigned)grid_blocks), dim3(kFwThreads), 0, s, g, several_producers, kept, kept_count,
                       FO, B, F, K, flags);
    return hipGetLastError();
}

}  // namespace dgn
