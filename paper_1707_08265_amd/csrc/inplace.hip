// In-place structures on the pruned graph (Sec. 2.4, Algorithm 3 of the paper).
//
// Algorithm 3 walks the nodes in order; a node not yet renamed becomes its own ancestor and hands that
// ancestor down while the current node has exactly one child.  On an acyclic graph the outcome does
// not depend on doing this one walk after the other: the nodes with exactly one child and their child
// form a forest of links p -> c, and the ancestor of v is the smallest id among the nodes from which v
// is reached over links, v included (that node cannot have been entered by an earlier walk, and
// neither can anything on its way to v).  That minimum is computed here by pointer doubling:
//   round k:  rename[J_k[u]] = min(rename[J_k[u]], rename[u]),  J_{k+1}[u] = J_k[J_k[u]]
// with J_0 = the link.  After round k every node has seen all nodes fewer than 2^(k+1) links upstream.
// rename[] is lowered in place with atomicMin (any value a round reads is an id that reaches the node,
// and at least as small as the value the round started with); the jump pointers are double buffered.
//
// Nodes are tensors; Child(x) = distinct tensors written by surviving operators that read x, where an
// operator survives when (K[o] & select) != 0.  "Exactly one child" is decided without building the
// sets: child[x] holds the only child seen so far and is set to "many" by whoever brings a second one.
//
// Only the two fills go over all tensors (100 M of them: 0.13 ms, the rate of a fill; 0.18 with 2 048 workgroups that walk them instead of
// a thread per 16 bytes, handed out in order); everything else follows the pruned
// graph: its nodes with links are listed when they are first offered a child, where a pass over all tensors looked for
// them before (0.17 ms).  456 000 kept operators with 1.5 M inputs on that graph, whole call: 0.65 -> 0.38 ms.
#include "common.h"

namespace dgn {

constexpr int kIpFillThreads = 256;
constexpr int kManyChildren = -2;                   // child[x]: -1 none yet, >= 0 the only child so far

// p[0..n) = -1, with 16-byte stores over the aligned bulk
__device__ __forceinline__ void fill_minus_one(int32_t *p, int64_t n, int64_t gtid, int64_t gsize)
{
    int64_t head = (int64_t)(((16 - ((uintptr_t)p & 15)) & 15) >> 2);
    if (head > n) head = n;
    if (gtid < head) p[gtid] = -1;
    int4 *bulk = reinterpret_cast<int4 *>(p + head);
    const int64_t quads = (n - head) >> 2;
    const int4 m = make_int4(-1, -1, -1, -1);
    for (int64_t i = gtid; i < quads; i += gsize) bulk[i] = m;
    const int64_t done = head + (quads << 2);
    if (gtid < n - done) p[done + gtid] = -1;
}

__global__ __launch_bounds__(kIpFillThreads) void k_inplace_init(int32_t *rename, int32_t *child, int64_t T,
                                                              int32_t *counters, int num_counters,
                                                              int64_t *renamed_count)
{
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t gsize = (int64_t)gridDim.x * blockDim.x;
    fill_minus_one(rename, T, gtid, gsize);
    fill_minus_one(child, T, gtid, gsize);
    if (blockIdx.x == 0) {
        if ((int)threadIdx.x < num_counters) counters[threadIdx.x] = 0;
        if (threadIdx.x == 0 && renamed_count) *renamed_count = 0;
    }
}

// The claimed nodes of a workgroup are gathered in LDS, so that the list's counter in memory is bumped once per workgroup and
// step, not once per wave (updates of one address take 11 ns each: a wave each would cost more than the pass itself).
// What finds no room goes to the list one wave at a time, so the room is for what a step of most graphs claims.
struct ClaimStage {
    int32_t *buf;                                   // [room]
    int room;
    int *count;                                     // claims of the workgroup since the last flush; past the room they
                                                    // went to the list one by one
    int32_t *list;
    int32_t *list_count;
};

// 64 operators, one per lane (valid lanes only): the tensors they touch become nodes of the graph (rename[x] = x), and each
// input learns its operator's output(s) as child.  child[x] only moves -1 -> id -> kManyChildren; the lane whose atomic
// moved it away from -1 claims x, to exactly one lane per node.
// The input edges of all lanes are spread evenly over the wave (prefix sum, then a running maximum over the marks where
// an operator's edges begin): an edge is a chain of dependent accesses -- id, child word, atomic --, and with an operator
// per lane a wave went through it as often as its operator with the most inputs asks for (0.25 -> 0.18 ms; what is left is
// about five scattered accesses per edge at the chip's rate for those).
template <RowForm kForm>
__device__ __forceinline__ void offer_children(const GraphView &g, bool valid, int64_t o, int32_t *rename, int32_t *child,
                                               int *s_mark, const ClaimStage &cs)
{
    constexpr int kNone = -1;                               // an operator without outputs offers nothing
    const int lane = lane_id();
    int eb = 0, deg = 0;
    int32_t offered = kNone;
    if (valid) {
        const int4 r = op_record<kForm>(g, (int32_t)o);
        eb = r.x;
        deg = r.y;
        const int n_out = kForm == kRun || r.w >= 0 ? r.w : -r.w;
        int lo = 0x7fffffff, hi = -1;
        for (int j = 0; j < n_out; ++j) {
            const int32_t u = kForm == kRun || r.w >= 0 ? r.z + j : g.out_idx[r.z + j];
            rename[u] = u;
            lo = min(lo, u);
            hi = max(hi, u);
        }
        if (n_out > 0) offered = lo == hi ? lo : kManyChildren;
    }
    const int incl = wave_incl_scan(deg), excl = incl - deg;
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    for (int w0 = 0; w0 < total; w0 += kWave) {             // wave-uniform
        s_mark[lane] = 0;
        __builtin_amdgcn_wave_barrier();
        if (deg > 0 && incl > w0 && excl < w0 + kWave) s_mark[max(excl - w0, 0)] = lane + 1;
        __builtin_amdgcn_wave_barrier();
        const int owner = max(wave_incl_max(s_mark[lane]) - 1, 0);
        __builtin_amdgcn_wave_barrier();
        const int o_eb = __shfl(eb, owner, kWave), o_excl = __shfl(excl, owner, kWave);
        const int32_t c = __shfl(offered, owner, kWave);
        bool claimed = false;
        int32_t x = 0;
        if (w0 + lane < total) {
            x = g.in_idx[o_eb + (w0 + lane - o_excl)];
            rename[x] = x;
            if (c == kManyChildren) {                       // two distinct children at once
                __hip_atomic_store(&child[x], kManyChildren, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else if (c != kNone) {
                const int32_t seen = child[x];              // (a stale value only costs an atomic)
                if (seen != c && seen != kManyChildren) {
                    const int32_t old = atomicCAS(&child[x], -1, c);
                    claimed = old == -1;
                    if (!claimed && old != c && old != kManyChildren)
                        __hip_atomic_store(&child[x], kManyChildren, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        const u64 cm = ballot64(claimed);
        if (cm) {
            int base = 0;
            if (lane == 0) base = atomicAdd(cs.count, __popcll(cm));
            const int pos = __builtin_amdgcn_readfirstlane(base) + __popcll(cm & lanemask_lt());
            if (claimed && pos < cs.room) cs.buf[pos] = x;
            const u64 om = ballot64(claimed && pos >= cs.room);
            if (om) {                                       // no room any more: straight into the list
                int at = 0;
                if (lane == 0) at = atomicAdd(cs.list_count, __popcll(om));
                at = __builtin_amdgcn_readfirstlane(at);
                if (claimed && pos >= cs.room) cs.list[at + __popcll(om & lanemask_lt())] = x;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
}

// Whole workgroup, after every step: the gathered claims go to the list once half of the room is taken, or at the end.
__device__ __forceinline__ void flush_claims(const ClaimStage &cs, int *s_base, bool last)
{
    __syncthreads();
    const int n = min(*cs.count, cs.room);
    __syncthreads();                                        // everyone has read the count before it changes again
    if (n == 0 || (n <= cs.room / 2 && !last)) return;    // the same in every thread
    if (threadIdx.x == 0) {
        *s_base = atomicAdd(cs.list_count, n);
        *cs.count = 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) cs.list[*s_base + i] = cs.buf[i];
    __syncthreads();
}

// Surviving operators can be a few percent of all: a wave reads 512 masks, packs the ids of the
// survivors into LDS and works on them 64 at a time, so that the dependent loads of the expansion
// run with all lanes busy.
//   Workgroups of 256 threads, with room for a claim per operator of a step; in one of 1 024, with room for every second, waves wait for each other and
// claims go to the list one wave at a time (4 096 graphs of 20 000, 49 M kept: 4.59 ms, 3.84 to 4.14 so; with half the large ones' room 7.41.  256 of 20 000: 312 us, 275;
// 50 M of a power law 455, 404; 800 000 in layers 155, 120).  Not for chains, whose operators read the same few graph inputs: the more waves
// go side by side, the more of them meet there (an RNN of 1 M: 176 us, with small workgroups 213; 200 000: 129, 133),
// nor where nobody knows (Meet::unknown).
constexpr int kMaskRounds = 8;                      // masks per lane and step
constexpr int kMaskThreads = 256, kChainThreads = 1024;
__host__ __device__ constexpr int mask_room(int threads) { return threads == kChainThreads ? 4096 : threads * kMaskRounds; }

template <RowForm kForm, int kThreads>
__global__ __launch_bounds__(kThreads) void k_inplace_children(GraphView g, const u64 *K, u64 select, int32_t *rename,
                                                                  int32_t *child, int32_t *list, int32_t *list_count)
{
    constexpr int kWaves = kThreads / kWave, kRoom = mask_room(kThreads);
    __shared__ int32_t s_ops[kWaves][kWave * (kMaskRounds + 1)];
    __shared__ int32_t s_claims[kRoom];
    __shared__ int s_mark[kWaves][kWave];
    __shared__ int s_count, s_base;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_count = 0;
    __syncthreads();
    const ClaimStage cs{s_claims, kRoom, &s_count, list, list_count};
    int32_t *ops = s_ops[wave];
    int count = 0;                                          // wave-uniform
    const int64_t step = (int64_t)kWave * kMaskRounds;
    const int64_t steps = ((int64_t)g.num_ops + step - 1) / step;
    const int64_t num_waves = (int64_t)gridDim.x * kWaves;
    for (int64_t st0 = (int64_t)blockIdx.x * kWaves; st0 < steps; st0 += num_waves) {      // whole workgroups stay in the loop
        const int64_t st = st0 + wave;
        u64 k[kMaskRounds];
#pragma unroll
        for (int r = 0; r < kMaskRounds; ++r) {
            const int64_t o = st * step + r * kWave + lane;
            k[r] = o < g.num_ops ? K[o] : 0;
        }
#pragma unroll
        for (int r = 0; r < kMaskRounds; ++r) {
            const bool kept = (k[r] & select) != 0;
            const u64 m = ballot64(kept);
            if (kept) ops[count + __popcll(m & lanemask_lt())] = (int32_t)(st * step + r * kWave + lane);
            count += __popcll(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        while (count >= kWave) {
            count -= kWave;
            offer_children<kForm>(g, true, ops[count + lane], rename, child, s_mark[wave], cs);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        flush_claims(cs, &s_base, false);
    }
    offer_children<kForm>(g, lane < count, lane < count ? ops[lane] : 0, rename, child, s_mark[wave], cs);
    flush_claims(cs, &s_base, true);
}

// The same from the list of kept operators that the prune wrote (ascending ids of the operators with K != 0):
// a pruned graph is a few percent of the recorded one, and the list spares the pass over all of K.  An entry
// whose mask misses `select` is skipped.  Workgroups are small, so that their number, not that of the workgroups on the chip, decides how long the
// last ones take (1.1 M operators of a power law with 2.8 M inputs: 190 us in workgroups of 1 024 threads, two and a little each, now 174).
//   Operators of chains and of a batch's graphs read the same few graph inputs, and all waves at once ask one after the other for the same
// line.  There a wave takes two times 64 entries one after the other, of long lists eight times: its later ones see that those inputs have
// several children already.  Whole pass, 1 024 threads and 64 entries each / 256 and 64 / 128 / 512: RNN of 1 M operators, 200 000 kept 313 / 442 /
// 259 / 163 us; 10 M, 515 000 kept 703 / 827 / 594 / 277; 46 000 kept 158 / 169 / 128 / 128, but of 500 000 with layers of 100 55 / 53 / 53 / 78; 40
// graphs of 300 000 1 930 / 2 050 / 2 260 / 1 240, 64 of them 2 370 / 2 660 / 3 030 / 1 890, 1 024 of 3 000 163 / 160 / 157 / 155, but 96 of 3 000 61 / 58 /
// 57 / 82, eight of 2 000 54 / 45 / 47 / 70.  Layers and power laws have no such inputs (50 M, 1 M kept, with the lists 641 us, with 128 entries 662).
// Where nobody knows, 128: an RNN of 1 M 223 / 221 / 175, 5 M of a power law 97 / 90 / 89, 500 layers of 400 72 / 69 / 72.
constexpr int kListThreads = 256, kListWaves = kListThreads / kWave, kListRoom = 2048;
constexpr int kListSomeRounds = 2, kListManyRounds = 8;
constexpr int64_t kListSome = (int64_t)1 << 15, kListManyOfChains = (int64_t)1 << 17, kListManyOfBatch = (int64_t)1 << 20, kListNever = (int64_t)1 << 62;
template <RowForm kForm>
__global__ __launch_bounds__(kListThreads) void k_inplace_children_list(GraphView g, const u64 *K, u64 select,
                                                                       const int32_t *kept_ops, const int64_t *kept_count, int64_t some,
                                                                       int64_t many, int32_t *rename, int32_t *child, int32_t *list,
                                                                       int32_t *list_count)
{
    __shared__ int32_t s_claims[kListRoom];
    __shared__ int s_mark[kListWaves][kWave];
    __shared__ int s_count, s_base;
    if (threadIdx.x == 0) s_count = 0;
    __syncthreads();
    const ClaimStage cs{s_claims, kListRoom, &s_count, list, list_count};
    const int64_t kept = kept_count[0];
    const int rounds = kept >= many ? kListManyRounds : kept >= some ? kListSomeRounds : 1;
    const int64_t tile = (int64_t)kListThreads * rounds, gsize = gridDim.x * tile;
    for (int64_t base = blockIdx.x * tile; base < kept; base += gsize) {       // whole workgroups stay in the loop
        const int64_t first = base + (int64_t)(threadIdx.x >> 6) * kWave * rounds + lane_id();
        for (int r = 0; r < rounds; ++r) {
            const int64_t i = first + r * kWave;
            const int32_t o = i < kept ? kept_ops[i] : 0;
            const bool valid = i < kept && (K[o] & select) != 0;
            offer_children<kForm>(g, valid, o, rename, child, s_mark[threadIdx.x >> 6], cs);
        }
        flush_claims(cs, &s_base, false);
    }
    flush_claims(cs, &s_base, true);
}

constexpr int kIpThreads = 1024;

// One doubling round over the claimed nodes.  J_0 is the child word itself (below zero: no link); the later pointers are
// kept for claimed nodes only, and child tells whether a node has one.  active[-1]: the round before left a pointer
// alive (first: there is none before).
__global__ __launch_bounds__(kIpThreads) void k_inplace_round(const int32_t *list, const int32_t *list_count, bool first,
                                                               const int32_t *child, const int32_t *Jcur, int32_t *Jnext,
                                                               int32_t *rename, int32_t *active, int64_t *renamed_count)
{
    __shared__ int s_more, s_newly;
    if (!first && active[-1] == 0) return;                  // (all pointers have run out: so has this round's)
    const int n = *list_count;
    const int gsize = gridDim.x * kIpThreads;
    if ((int)(blockIdx.x * kIpThreads) >= n) return;
    if (threadIdx.x == 0) s_more = s_newly = 0;
    __syncthreads();
    bool more = false;
    int newly = 0;
    for (int i = blockIdx.x * kIpThreads + threadIdx.x; i < n; i += gsize) {
        const int32_t u = list[i];
        const int32_t v = Jcur[u];
        int32_t next = -1;
        if (v >= 0) {
            const int32_t a = rename[u], link = child[v];
            const int32_t j = first ? link : Jcur[v];       // (not a pointer when v has no link)
            const int32_t old = atomicMin(&rename[v], a);
            if (old == v && a < v) ++newly;                 // v carried its own name until now
            if (link >= 0) next = j;
        }
        Jnext[u] = next;
        more |= next >= 0;
    }
    const u64 mm = ballot64(more);
    const int wnew = wave_sum(newly);
    if (lane_id() == 0) {                                   // one update of each word in memory per workgroup
        if (mm) s_more = 1;
        if (wnew) atomicAdd(&s_newly, wnew);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_more) *active = 1;
        if (s_newly && renamed_count) atomicAdd((u64 *)renamed_count, (u64)s_newly);
    }
}

size_t inplace_scratch_bytes(int64_t T)
{
    const size_t t = (size_t)(T > 0 ? T : 1);
    return 4 * ((t * 4 + 255) & ~(size_t)255) + 256;
}

InplaceBuffers inplace_buffers(void *scratch, int64_t T)
{
    const size_t t = (size_t)(T > 0 ? T : 1);
    char *p = static_cast<char *>(scratch);
    InplaceBuffers b;
    b.child = reinterpret_cast<int32_t *>(p); p += (t * 4 + 255) & ~(size_t)255;
    b.J[0] = reinterpret_cast<int32_t *>(p); p += (t * 4 + 255) & ~(size_t)255;
    b.J[1] = reinterpret_cast<int32_t *>(p); p += (t * 4 + 255) & ~(size_t)255;
    b.list = reinterpret_cast<int32_t *>(p); p += (t * 4 + 255) & ~(size_t)255;
    b.counters = reinterpret_cast<int32_t *>(p);
    return b;
}

hipError_t launch_inplace_setup(const GraphView &g, const u64 *K, u64 select, const int32_t *kept_ops,
                                const int64_t *kept_count, int32_t *rename, int64_t *renamed_count,
                                const InplaceBuffers &b, Meet meet, int grid_blocks, hipStream_t s)
{
    const int64_t T = g.num_tensors, P = g.num_ops;
    // fills: a thread per 16 bytes and array; the other passes: as many threads as the chip holds
    const int64_t nb = (T + kIpFillThreads * 4 - 1) / (kIpFillThreads * 4);
    hipLaunchKernelGGL(k_inplace_init, dim3((unsigned)(nb < 1 ? 1 : nb)), dim3(kIpFillThreads), 0, s, rename, b.child, T, b.counters,
                       kInplaceMaxRounds + 1, renamed_count);
    const RowForm rows = rows_of(g);
    const bool chains = meet == Meet::chains || meet == Meet::unknown;
    const int threads = kept_ops ? kListThreads : chains ? kChainThreads : kMaskThreads;
    int64_t blocks = (P + threads - 1) / threads;
    if (blocks > grid_blocks * 256 / threads) blocks = grid_blocks * 256 / threads;
    if (P > 0 && kept_ops) {
        auto k = rows == kRun ? k_inplace_children_list<kRun> : rows == kRecords ? k_inplace_children_list<kRecords> : k_inplace_children_list<kFirst>;
        hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), 0, s, g, K, select, kept_ops, kept_count,
                           meet == Meet::nowhere ? kListNever : kListSome,
                           meet == Meet::chains ? kListManyOfChains : meet == Meet::batch ? kListManyOfBatch : kListNever, rename, b.child, b.list, b.counters);
    } else if (P > 0) {
        auto k = rows == kRun       ? chains ? k_inplace_children<kRun, kChainThreads> : k_inplace_children<kRun, kMaskThreads>
                 : rows == kRecords ? chains ? k_inplace_children<kRecords, kChainThreads> : k_inplace_children<kRecords, kMaskThreads>
                                    : k_inplace_children<kFirst, kMaskThreads>;            // (batches)
        hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(threads), 0, s, g, K, select, rename, b.child, b.list, b.counters);
    }
    return hipGetLastError();
}

hipError_t launch_inplace_round(int round, int32_t *rename, int64_t *renamed_count, const InplaceBuffers &b,
                                int grid_blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_inplace_round, dim3((unsigned)(grid_blocks / 4)), dim3(kIpThreads), 0, s, b.list, b.counters,
                       round == 0, b.child, round == 0 ? b.child : b.J[round & 1], b.J[(round & 1) ^ 1], rename,
                       b.counters + 1 + round, renamed_count);
    return hipGetLastError();
}

}  // namespace dgn
