// Stable sorts of (int32 key, int32 value) pairs for the CSR builder: an LSD radix sort of at most 9 bits per pass, and rows by way
// of buckets, which sorts the high bits that way and the rest inside a workgroup (second half of this file).
//
// Per pass: (1) digit counts per tile of 8 192 keys, already summed inside groups of 16 tiles, and each group's totals;
// (2) a small scan of the groups' totals; (3) a scatter in which every wave ranks its keys against the keys of its
// lower lanes and earlier rounds (ballot "match" masks): keys of one tile are visited in their stored order, so
// equal keys keep their relative order.  The tile is sorted inside LDS first, so that it leaves in one run per digit.
// Only the significant key bits are sorted.  (A whole sort of 26 bits in eight bits per pass and four passes: 9 % slower than three
// of nine; a pass with 512 digits costs more than one with 256, because a tile then leaves in runs half as long and the ranking
// takes a step more, but not a third more.)
//
// What a pass costs, per 32 M pairs: counting 27 us (the keys once, at the rate of a copy), the scan 5, the scatter 131 us = 3.9 TB/s
// of 16 bytes per pair with eight bits (126 with seven: it is memory that bounds it).  The scatter's time went, in turn, to
// the write-back of half-written cache lines (fixed by giving each die a contiguous range of tiles), to one cache
// line per digit and tile for the slot table (fixed by the tile-major tables), and to the vector instructions of the
// ranking (halved by the three-input bit operation and longer tiles).
#include "common.h"

namespace dgn {

constexpr int kMaxRadixBits = 9;
constexpr int kSortThreads = 1024;                      // threads of a scattering workgroup; the first 2^bits of them
                                                        // also keep the books of one digit each
constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kSortRounds = 8;                          // keys per lane
constexpr int kSortTile = kSortThreads * kSortRounds;   // keys per workgroup

template <int kBits> __device__ __forceinline__ int digit_of(int32_t key, int shift)
{
    return ((uint32_t)key >> shift) & ((1 << kBits) - 1);
}

// The first output slot of a tile's keys with digit d is the number of keys that sort before them: all keys with a
// smaller digit, and the keys with digit d of earlier tiles.  It is kept in two tables, both tile-major (a row of
// kRadix words per tile or per group of tiles), so that the workgroup that counts a tile and the one that scatters it
// both touch one contiguous row -- a digit-major table costs the scatter one cache line per digit and tile, a fifth of
// all the cache lines it asks for:
//   table[tile][d]   keys with digit d in the earlier tiles of the tile's group of kHistTiles consecutive tiles,
//   totals[group][d] first the group's keys with digit d, then (k_col_apply) the keys with a smaller digit anywhere plus
//                    those with digit d in earlier groups.
//   sums[chunk][d]   the keys with digit d in a chunk of consecutive groups, added up by the groups; two of them, so that one pass clears
//                    the next one's.
constexpr int kHistTiles = 16;
constexpr int kColChunks = 64;              // the groups are scanned in up to this many chunks of consecutive groups

constexpr int kHistThreads = 1024;

// Adds the digits of a thread's kPer neighbouring keys to a tile's counts.  In a list that is nearly in order the lanes of a wave
// mostly have the same digit of the high bits (two of them, where two such lists are interleaved), and an atomic per key has
// all of them wait for each other: 4 M edges in order but for one took 100 us, in no order 15.  So where many lanes have the digit of
// the one in the middle, a thread adds up what it has of its first digit and of the next other one, and a wave of one digit alone adds
// once: 20 us; builds of two recordings one behind the other, 200 000 operators 305 -> 151, 2 M 637 -> 309, 10 M 1 221 -> 921.
constexpr int kSameDigit = 8;               // lanes
template <int kPer> __device__ __forceinline__ void count_digits(int *hist, const int (&d)[kPer], int valid)
{
    const int same = __popcll(ballot64(d[0] == __builtin_amdgcn_readlane(d[0], kWave / 2)));
    if (same < kSameDigit) {
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (q < valid) atomicAdd(&hist[d[q]], 1);
        return;
    }
    int count = 0, other = d[0], others = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        count += q < valid && d[q] == d[0];
        other = other == d[0] && q < valid ? d[q] : other;
    }
    if (same == kWave && ballot64(count < kPer) == 0) {
        if (lane_id() == 0) atomicAdd(&hist[d[0]], kWave * kPer);
        return;
    }
    if (count) atomicAdd(&hist[d[0]], count);
    if (other == d[0]) return;
#pragma unroll
    for (int q = 0; q < kPer; ++q) others += q < valid && d[q] == other;
    atomicAdd(&hist[other], others);
    if (count + others < valid) {
#pragma unroll
        for (int q = 0; q < kPer; ++q)
            if (q < valid && d[q] != d[0] && d[q] != other) atomicAdd(&hist[d[q]], 1);
    }
}

template <int kBits>
__global__ __launch_bounds__(kHistThreads) void k_sort_hist(const int32_t *keys, int64_t n, int shift, int32_t *table,
                                                                     int32_t *totals, int32_t *sums, int per_chunk,
                                                                     uint32_t num_rows, int32_t *status)
{
    constexpr int kRadix = 1 << kBits, kThreads = kHistThreads;
    __shared__ int hist[kHistTiles][kRadix];
    for (int i = threadIdx.x; i < kHistTiles * kRadix; i += kThreads) (&hist[0][0])[i] = 0;
    __syncthreads();
    const int64_t tile0 = (int64_t)blockIdx.x * kHistTiles;
    uint32_t most = 0;                                       // the largest key, for the check (status not NULL)
    const bool wide = (reinterpret_cast<uintptr_t>(keys) & 15) == 0;
    constexpr int kPerThread = kSortTile / kThreads;         // keys of a tile that one thread counts
    static_assert(kPerThread % 4 == 0, "a thread counts whole 16-byte groups of keys");
    // the order inside a tile does not matter for its counts: a thread takes neighbouring keys, and asks for the next tile's ahead
    int32_t next[kPerThread];
    auto first_of = [&](int t) { return (tile0 + t) * kSortTile + (int64_t)threadIdx.x * kPerThread; };
    auto ask = [&](int64_t i) {
        if (wide && i + kPerThread <= n) {
#pragma unroll
            for (int q = 0; q < kPerThread; q += 4) {
                const int4 v = *reinterpret_cast<const int4 *>(keys + i + q);
                next[q] = v.x; next[q + 1] = v.y; next[q + 2] = v.z; next[q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < kPerThread; ++q) next[q] = i + q < n ? keys[i + q] : 0;
        }
    };
    ask(first_of(0));
    for (int t = 0; t < kHistTiles; ++t) {
        const int64_t i = first_of(t);
        if (i - (int64_t)lane_id() * kPerThread >= n) break;             // whole waves stay in the loop
        int d[kPerThread];
#pragma unroll
        for (int q = 0; q < kPerThread; ++q) {
            most = max(most, (uint32_t)next[q]);
            d[q] = digit_of<kBits>(next[q], shift);
        }
        if (t + 1 < kHistTiles) ask(first_of(t + 1));
        count_digits(hist[t], d, (int)min(max(n - i, (int64_t)0), (int64_t)kPerThread));
    }
    __syncthreads();
    if (status && ballot64(most >= num_rows) != 0 && lane_id() == 0) atomicOr(status, kErrIdRange);
    // the table has a row for each of the group's kHistTiles tiles, also past the last tile
    const bool keeps_digit = threadIdx.x < kRadix;
    int run = 0;
    if (keeps_digit) {
        int32_t *row = table + tile0 * kRadix + threadIdx.x;
#pragma unroll
        for (int t = 0; t < kHistTiles; ++t) {
            row[t * kRadix] = run;
            run += hist[t][threadIdx.x];
        }
    }
    if (gridDim.x == 1) {                                    // a list of one group: k_col_apply has nothing to add up but the digits
        __shared__ int s_wtot[kThreads / kWave];
        const int incl = wave_incl_scan(run);
        if (lane_id() == kWave - 1) s_wtot[threadIdx.x >> 6] = incl;
        __syncthreads();
        int first = incl - run;
        for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) first += s_wtot[w];
        if (keeps_digit) totals[threadIdx.x] = first;
        return;
    }
    if (!keeps_digit) return;
    totals[(int64_t)blockIdx.x * kRadix + threadIdx.x] = run;
    if (run) atomicAdd(&sums[(int64_t)(blockIdx.x / per_chunk) * kRadix + threadIdx.x], run);
}

// Exclusive scan of totals[group][d] in the order (d, group): a workgroup per chunk of groups, a thread per digit.  Every
// workgroup works out its chunk's start by itself from all chunks' sums (the columns' totals scanned across the digits, plus
// the earlier chunks of the column) and then walks down its rows.
// (every walk down a column asks for kColBatch rows at a time: one row per round trip would leave this small
// kernel waiting for memory most of its time)
constexpr int kColBatch = 8;

template <int kBits>
__global__ __launch_bounds__(1 << kBits) void k_col_apply(int32_t *totals, int64_t groups, int per_chunk, const int32_t *sums,
                                                          int chunks, int32_t *next_sums)
{
    constexpr int kRadix = 1 << kBits, kDigitWaves = kRadix / kWave;
    __shared__ int s_wtot[kDigitWaves];
    const int d = threadIdx.x, lane = lane_id(), wave = threadIdx.x >> 6;
    int v[kColChunks];                                       // the whole column, in registers
#pragma unroll
    for (int c = 0; c < kColChunks; ++c) v[c] = c < chunks ? sums[c * kRadix + d] : 0;
    next_sums[blockIdx.x * kRadix + d] = 0;
    int col = 0, earlier = 0;
#pragma unroll
    for (int c = 0; c < kColChunks; ++c) {
        if (c < (int)blockIdx.x) earlier += v[c];
        col += v[c];
    }
    const int incl = wave_incl_scan(col);
    if (lane == kWave - 1) s_wtot[wave] = incl;
    __syncthreads();
    int run = incl - col + earlier;                          // keys with a smaller digit, and of this one in earlier chunks
#pragma unroll
    for (int w = 0; w < kDigitWaves; ++w)
        if (w < wave) run += s_wtot[w];
    const int64_t g0 = (int64_t)blockIdx.x * per_chunk;
    const int rows = (int)min((int64_t)per_chunk, groups - g0);
    int32_t *column = totals + g0 * kRadix + d;
    for (int r = 0; r < rows; r += kColBatch) {
        int x[kColBatch];
#pragma unroll
        for (int j = 0; j < kColBatch; ++j) x[j] = r + j < rows ? column[(r + j) * kRadix] : 0;
#pragma unroll
        for (int j = 0; j < kColBatch; ++j) {
            if (r + j < rows) column[(r + j) * kRadix] = run;
            run += x[j];
        }
    }
}

// The lanes that hold a key (valid) with the same digit as this one: how many in all, and how many of them are lower lanes.
// others = the lanes whose digit differs from this lane's in some bit (or that hold no key).  For bit b, m =
// the lanes that have it set and e = this lane's own bit spread over a word: m ^ e marks the lanes that
// differ in b.  Kept as two 32-bit halves and as the complement of the usual "peers" mask, this is four
// vector instructions per bit; a sort's time is mostly vector instructions, and most of them are these.
template <int kBits>
__device__ __forceinline__ void match_digit(int d, bool valid, uint32_t lt_lo, uint32_t lt_hi, int &before, int &same)
{
    const u64 held = ballot64(valid);
    uint32_t others_lo = ~(uint32_t)held, others_hi = ~(uint32_t)(held >> 32);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
        int32_t e = __builtin_amdgcn_sbfe(d, b, 1);                     // -1 if bit b of d is set, else 0
        asm("" : "+v"(e));                                              // (compare e itself, not d shifted once more)
        const u64 m = ballot64(e != 0);
        others_lo = or_of_xor(others_lo, (uint32_t)m, (uint32_t)e);
        others_hi = or_of_xor(others_hi, (uint32_t)(m >> 32), (uint32_t)e);
    }
    before = lane_id() - (__popc(others_lo & lt_lo) + __popc(others_hi & lt_hi));
    same = kWave - (__popc(others_lo) + __popc(others_hi));
}

// (eight waves per SIMD: two workgroups of 1 024 threads per CU, which caps the kernel at 64 vector registers)
template <int kBits>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
void k_sort_scatter(const int32_t *keys, const int32_t *vals, int32_t *keys_out, int32_t *vals_out, int64_t n, int shift,
                    const int32_t *table, const int32_t *totals, int64_t num_tiles)
{
    constexpr int kRadix = 1 << kBits, kDigitWaves = kRadix / kWave;
    // Workgroups go to the chip's eight dies in turn, each with a second-level cache of its own.  Neighbouring tiles
    // write neighbouring runs of the output (a run is shorter than a cache line), so a die takes a contiguous eighth
    // of the tiles and the two halves of a line meet in one cache.
    const int64_t per_die = (num_tiles + 7) >> 3;
    const int64_t tile = (int64_t)(blockIdx.x & 7) * per_die + (blockIdx.x >> 3);
    if (tile >= num_tiles) return;
    // first output slot of this tile's keys with digit threadIdx.x: asked for now, needed after the ranking
    const bool keeps_digit = threadIdx.x < kRadix;
    int32_t first_slot = 0;
    if (keeps_digit) first_slot = table[tile * kRadix + threadIdx.x] + totals[tile / kHistTiles * kRadix + threadIdx.x];
    // the per-wave digit counts are dead once every key knows its slot in the sorted tile: the tile takes their place
    __shared__ int32_t s_raw[2 * kSortTile];
    static_assert(kSortWaves * kRadix <= 2 * kSortTile, "the counts fit into the tile's storage");
    int (*wcount)[kRadix] = reinterpret_cast<int (*)[kRadix]>(s_raw);
    int32_t *s_keys = s_raw, *s_vals = s_raw + kSortTile;
    __shared__ int s_delta[kRadix];          // global slot of a key = its slot in the locally sorted tile + this
    __shared__ int s_wtot[kDigitWaves];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < kSortWaves * kRadix; i += kSortThreads) (&wcount[0][0])[i] = 0;
    __syncthreads();

    // wave w owns kSortRounds * 64 consecutive keys of the tile, visited 64 at a time
    const int64_t tbase = tile * kSortTile;
    const int count = (int)min((int64_t)kSortTile, n - tbase);          // keys of this tile
    const int32_t *tile_keys = keys + tbase, *tile_vals = vals + tbase;
    const int wofs = wave * (kSortRounds * kWave) + lane;
    int32_t key[kSortRounds], val[kSortRounds];
    int rank[kSortRounds];
    const u64 lt = lanemask_lt();
    const uint32_t lt_lo = (uint32_t)lt, lt_hi = (uint32_t)(lt >> 32);
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        const int i = wofs + r * kWave;
        const bool valid = i < count;
        key[r] = valid ? tile_keys[i] : 0;
        val[r] = valid ? tile_vals[i] : 0;
        const int d = digit_of<kBits>(key[r], shift);
        int before, same;
        match_digit<kBits>(d, valid, lt_lo, lt_hi, before, same);
        // lanes with the same digit read the running count, then their first lane bumps it
        const int c = wcount[wave][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) wcount[wave][d] = c + same;
        __builtin_amdgcn_wave_barrier();
        rank[r] = c + before;
    }
    __syncthreads();
    {   // digit d (one per thread): per-wave counts -> first slot of each wave's keys in the locally sorted tile
        const int d = threadIdx.x;
        int cnt = 0, incl = 0;
        if (keeps_digit) {
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) cnt += wcount[w][d];
            incl = wave_incl_scan(cnt);
            if (lane == kWave - 1) s_wtot[wave] = incl;
        }
        __syncthreads();
        if (keeps_digit) {
            int lbase = incl - cnt;
#pragma unroll
            for (int w = 0; w < kDigitWaves; ++w)
                if (w < wave) lbase += s_wtot[w];
            s_delta[d] = first_slot - lbase;
            int run = lbase;
#pragma unroll
            for (int w = 0; w < kSortWaves; ++w) {
                const int c = wcount[w][d];
                wcount[w][d] = run;
                run += c;
            }
        }
    }
    __syncthreads();
    // sort the tile inside LDS, so that the global writes below go out in long contiguous runs per digit
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) rank[r] += wcount[wave][digit_of<kBits>(key[r], shift)];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortRounds; ++r) {
        if (wofs + r * kWave < count) {
            s_keys[rank[r]] = key[r];
            s_vals[rank[r]] = val[r];
        }
    }
    __syncthreads();
    for (int li = threadIdx.x; li < count; li += kSortThreads) {
        const int32_t k = s_keys[li];
        const int pos = li + s_delta[digit_of<kBits>(k, shift)];
        keys_out[pos] = k;
        vals_out[pos] = s_vals[li];
    }
}

static inline int64_t sort_tiles(int64_t n) { return (n + kSortTile - 1) / kSortTile; }
static inline int64_t sort_groups(int64_t tiles) { return (tiles + kHistTiles - 1) / kHistTiles; }

// layout of tmp: keyA[n] valA[n] keyB[n] valB[n] table[groups*kHistTiles][radix] totals[groups][radix]
// sums[2][kColChunks][radix]
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t sort_tmp_bytes(int64_t n)
{
    constexpr size_t kRadix = 1 << kMaxRadixBits;
    const int64_t groups = sort_groups(sort_tiles(n));
    return 4 * align256((size_t)n * 4) + align256((size_t)(groups * kHistTiles) * kRadix * 4) +
           align256((size_t)groups * kRadix * 4) + 2 * align256((size_t)kColChunks * kRadix * 4);
}

// Where a sort keeps what: two buffers of pairs and the tables of a pass.
struct SortTmp {
    int32_t *keys[2], *vals[2], *table, *totals, *sums;
    size_t table_bytes;
};

static SortTmp sort_tmp(void *tmp, int64_t n)
{
    constexpr size_t kRadix = 1 << kMaxRadixBits;
    const int64_t groups = sort_groups(sort_tiles(n));
    char *p = static_cast<char *>(tmp);
    auto take = [&](size_t bytes) {
        int32_t *r = reinterpret_cast<int32_t *>(p);
        p += align256(bytes);
        return r;
    };
    SortTmp t;
    for (int i = 0; i < 2; ++i) {
        t.keys[i] = take((size_t)n * 4);
        t.vals[i] = take((size_t)n * 4);
    }
    t.table_bytes = (size_t)(groups * kHistTiles) * kRadix * 4;
    t.table = take(t.table_bytes);
    t.totals = take((size_t)groups * kRadix * 4);
    t.sums = take(2 * (size_t)kColChunks * kRadix * 4);
    return t;
}

// `passes` stable passes over the key bits from `low` on, kBits at a time.  keys_out / vals_out: where the last one leaves the
// pairs, or NULL: in t.keys / t.vals[(passes - 1) & 1].  status (or NULL): kErrIdRange if a key is none of the num_rows rows.
template <int kBits>
static hipError_t sort_passes(const int32_t *keys_in, const int32_t *vals_in, int32_t *keys_out, int32_t *vals_out, int64_t n,
                              int low, int passes, const SortTmp &t, hipStream_t s, int64_t num_rows = 0, int32_t *status = nullptr)
{
    constexpr int kRadix = 1 << kBits;
    const int64_t tiles = sort_tiles(n), groups = sort_groups(tiles);
    const int per_chunk = (int)((groups + kColChunks - 1) / kColChunks);
    const int chunks = (int)((groups + per_chunk - 1) / per_chunk);
    const unsigned scatter_grid = (unsigned)(((tiles + 7) >> 3) << 3);
    int32_t *sums[2] = {t.sums, t.sums + kColChunks * kRadix};
    FillRegion clr[1] = {{sums[0], (size_t)chunks * kRadix * sizeof(int32_t)}};
    hipError_t e = groups > 1 ? launch_clear(clr, 1, s) : hipSuccess;
    if (e != hipSuccess) return e;
    const int32_t *ksrc = keys_in, *vsrc = vals_in;
    for (int pass = 0; pass < passes; ++pass) {
        const bool last = pass == passes - 1;
        const int shift = low + pass * kBits;
        int32_t *kdst = last && keys_out ? keys_out : t.keys[pass & 1];
        int32_t *vdst = last && vals_out ? vals_out : t.vals[pass & 1];
        hipLaunchKernelGGL(k_sort_hist<kBits>, dim3((unsigned)groups), dim3(kHistThreads), 0, s, ksrc, n, shift, t.table,
                           t.totals, sums[pass & 1], per_chunk, (uint32_t)num_rows, pass == 0 ? status : nullptr);
        if (groups > 1)
            hipLaunchKernelGGL(k_col_apply<kBits>, dim3(chunks), dim3(kRadix), 0, s, t.totals, groups, per_chunk,
                               sums[pass & 1], chunks, sums[(pass & 1) ^ 1]);
        hipLaunchKernelGGL(k_sort_scatter<kBits>, dim3(scatter_grid), dim3(kSortThreads), 0, s, ksrc, vsrc, kdst, vdst, n, shift,
                           t.table, t.totals, tiles);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        ksrc = kdst;
        vsrc = vdst;
    }
    return hipSuccess;
}

static int sort_pass_count(int key_bits) { return (key_bits + kMaxRadixBits - 1) / kMaxRadixBits; }

hipError_t launch_sort_pairs(const int32_t *keys_in, const int32_t *vals_in, int32_t *keys_out,
                             int32_t *vals_out, int64_t n, int key_bits, void *tmp, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    if (key_bits < 1) key_bits = 1;
    const int passes = sort_pass_count(key_bits);
    const SortTmp t = sort_tmp(tmp, n);
    return key_bits <= 8 * passes ? sort_passes<8>(keys_in, vals_in, keys_out, vals_out, n, 0, passes, t, s)
                                  : sort_passes<9>(keys_in, vals_in, keys_out, vals_out, n, 0, passes, t, s);
}

// ------------------------------------------------------------------------------------------------
// rows from a list in no order
//
// The adjacency needs the rows, not the sorted keys: passes as above bring the pairs into buckets of up to 512 neighbouring
// rows only (the high bits of the key), and one workgroup per bucket ranks what is left of the key in LDS and writes the
// bucket's rows and row pointers: a pass over memory less, no keys written at the end, and no pass that reads them again.  For
// outputs the same workgroup writes the rows by tensor, which took two more
// passes.  32 M input edges of 12 M operators: 530 us sorted as a whole, 475 so; their 25 M outputs 700 -> 455; the whole build
// 1 430 -> 1 055 us.  10 000 operators: 181 -> 135, 30 000: 220 -> 143, 500 000: 400 -> 190, 50 M: 5 390 -> 3 940.
//
// The last step takes 118 us for those 32 M pairs (440 MB), 177 for the outputs (590 MB; 226 while it wrote records and producer words as well): memory.  It was 205 with workgroups of 1 024
// threads, eleven bits of the key and two passes inside LDS (barriers, and vector instructions of the second pass), 156 with
// 256 threads and two passes.
// ------------------------------------------------------------------------------------------------
constexpr int kRowRounds = 8;                           // pairs per thread
template <int kThreads> struct Rows {
    static constexpr int kWaves = kThreads / kWave, kTile = kThreads * kRowRounds;      // pairs that a workgroup holds at a time
    static constexpr int kBits = kThreads == 256 ? 9 : 10, kRows = 1 << kBits;          // rows of a bucket, at most
    static_assert(kRows == 2 * kThreads, "two rows per thread");
};
// A bucket of more than a tile is done a tile after the other by its workgroup; one of more than kSerialTiles (an operator with very
// many inputs, say) by as many workgroups as it has tiles, in a launch of its own: any number of them, of any size.
constexpr int kSerialTiles = 8, kBigBlocks = 1024;
constexpr int kRowFillPercent = 75;                     // of a tile, on average, at most

// starts[b] = first position with a key of bucket b or above, big = the buckets of more than `most` pairs (fewer than max_big); four lanes
// per bucket probe a quarter of what is left each.
constexpr int kProbes = 4;
__global__ __launch_bounds__(256) void k_bucket_starts(const int32_t *keys, int32_t n, int row_bits, int32_t buckets, int32_t most,
                                                        int32_t *starts, int32_t *big, int32_t max_big, int32_t *num_big, int32_t *status)
{
    const int64_t thread = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // For the kernels behind this one, which add to status[0] themselves: all waves of a workgroup have to read the same here.
    if (thread == 0 && (status[0] & kErrIdRange)) status[kStatusNoRows] = 1;
    const int32_t b = (int32_t)min(thread / kProbes, (int64_t)buckets);
    const int probe = threadIdx.x & (kProbes - 1), group = lane_id() & ~(kProbes - 1);
    int32_t lo = 0, hi = b == buckets ? 0 : n;              // the answer is in [lo, hi]
    while (ballot64(hi > lo)) {                             // whole waves stay in the loop
        const int32_t step = (int32_t)(((int64_t)hi - lo + kProbes - 1) / kProbes);
        const int64_t at = (int64_t)lo + (int64_t)probe * step;
        const bool below = at < hi && (keys[at] >> row_bits) < b;
        const int c = __popcll((ballot64(below) >> group) & ((1 << kProbes) - 1));      // the keys ascend by bucket: the first c are below
        if (c > 0) {
            const int64_t after = (int64_t)lo + (int64_t)c * step;
            hi = (int32_t)min((int64_t)hi, after);
            lo = (int32_t)(after - step) + 1;
        } else {
            hi = lo;                                        // (lo itself is not below)
        }
    }
    if (b == buckets) lo = n;
    if (probe == 0) {
        starts[b] = lo;
        if (b < buckets && (int64_t)lo + most < n && (keys[lo + most] >> row_bits) == b) {
            const int at = atomicAdd(num_big, 1);
            if (at < max_big) big[at] = b;                  // (more only of keys that are no rows, and then nothing is made of them)
        }
    }
}

// The pairs of a tile in registers, ranked: rank[r] = keys of the same row before this one among those of its wave, counted in
// `count` (per wave, two neighbouring rows to a word).  Whole workgroup; ends with a barrier.
struct TilePairs {
    int row[kRowRounds], rank[kRowRounds];
    int32_t val[kRowRounds];
    int rounds, first;                                      // a wave owns 64 * rounds consecutive places of the tile
};

template <int kThreads>
__device__ __forceinline__ void rank_tile(const int32_t *keys, const int32_t *vals, int m, int32_t row0, int row_mask, int32_t num_tensors,
                                          uint32_t (*count)[Rows<kThreads>::kRows / 2], TilePairs &p, bool &bad)
{
    using R = Rows<kThreads>;
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const u64 lt = lanemask_lt();
    const uint32_t lt_lo = (uint32_t)lt, lt_hi = (uint32_t)(lt >> 32);
    uint16_t *const mine = reinterpret_cast<uint16_t *>(count[wave]);
    p.rounds = (m + kThreads - 1) / kThreads;
    p.first = wave * p.rounds * kWave + lane;
#pragma unroll
    for (int r = 0; r < kRowRounds; ++r) {
        const int i = p.first + r * kWave;
        const bool valid = r < p.rounds && i < m;
        p.row[r] = valid ? (keys[i] - row0) & row_mask : 0;
        p.val[r] = valid ? vals[i] : 0;
        bad |= (uint32_t)p.val[r] >= (uint32_t)num_tensors;
    }
#pragma unroll
    for (int w = 0; w < R::kWaves; ++w) count[w][threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRowRounds; ++r) {
        if (r >= p.rounds) break;                                           // (the same in every lane)
        const bool valid = p.first + r * kWave < m;
        int before, same;
        match_digit<R::kBits>(p.row[r], valid, lt_lo, lt_hi, before, same);
        const int c = mine[p.row[r]];
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) mine[p.row[r]] = (uint16_t)(c + same);
        __builtin_amdgcn_wave_barrier();
        p.rank[r] = c + before;
    }
    __syncthreads();
}

// Exclusive sum over the rows of a bucket, two of them per thread.  Whole workgroup; one barrier.
template <int kThreads>
__device__ __forceinline__ int row_scan(int both, int *s_wtot)
{
    const int wave = threadIdx.x >> 6, incl = wave_incl_scan(both);
    if (lane_id() == kWave - 1) s_wtot[wave] = incl;
    __syncthreads();
    int first = incl - both;
#pragma unroll
    for (int w = 0; w < Rows<kThreads>::kWaves; ++w)
        if (w < wave) first += s_wtot[w];
    return first;
}

// Adds up the counts of the waves: every wave's count becomes the place (from first[0], first[1] on) of its keys of the row.  v0, v1: the
// workgroup's counts of this thread's two rows.  Ends with a barrier.
template <int kThreads, typename First>
__device__ __forceinline__ void place_rows(uint32_t (*count)[Rows<kThreads>::kRows / 2], int &v0, int &v1, First first)
{
    using R = Rows<kThreads>;
    uint32_t sum = 0, earlier[R::kWaves];                                   // (no half of a word exceeds a tile: no carries)
#pragma unroll
    for (int w = 0; w < R::kWaves; ++w) {
        earlier[w] = sum;
        sum += count[w][threadIdx.x];
    }
    v0 = (int)(sum & 0xffff);
    v1 = (int)(sum >> 16);
    const uint32_t at = first(v0, v1);
#pragma unroll
    for (int w = 0; w < R::kWaves; ++w) count[w][threadIdx.x] = at + earlier[w];
    __syncthreads();
}

// How often the rows of a bucket occur among n keys.  Most may be of one row: its lanes add together.  Whole workgroup; the counts are
// zero before; ends with a barrier.
template <int kThreads>
__device__ __forceinline__ void count_rows(const int32_t *keys, int32_t n, int32_t row0, int row_mask, int *s_rows)
{
    for (int32_t i0 = threadIdx.x; i0 - lane_id() < n; i0 += kThreads * kRowRounds) {     // (whole waves)
        int row[kRowRounds];
#pragma unroll
        for (int r = 0; r < kRowRounds; ++r) row[r] = i0 + r * kThreads < n ? (keys[i0 + r * kThreads] - row0) & row_mask : -1;
#pragma unroll
        for (int r = 0; r < kRowRounds; ++r) {
            const int most = __builtin_amdgcn_readfirstlane(row[r]);
            const u64 m = ballot64(row[r] == most);
            if (most < 0) break;                            // (the same in every lane)
            if (lane_id() == 0) atomicAdd(&s_rows[most], __popcll(m));
            else if (row[r] >= 0 && row[r] != most) atomicAdd(&s_rows[row[r]], 1);
        }
    }
    __syncthreads();
}

// Big buckets are done in groups of tiles, a workgroup each: one launch counts every group's rows, the next adds up the groups before
// its own and goes through its tiles one after the other.  With few tiles to a group there are many groups to be added up, with
// many little is done at a time: the tiles of a group are 1 up to 64 tiles, 2 up to 256, and so on.  Shuffled builds of 10 M operators, 70
// of them with 17 000 inputs: 745 us, of 200 000 1 058, one of 4 M 854, of 60 M 2 024 (lists sorted as a whole: 939, 1 345, 1 140 and
// 2 375).
template <int kThreads> struct BigBucket {
    int32_t tiles, group, groups;
    __device__ __forceinline__ explicit BigBucket(int32_t pairs)
    {
        tiles = (pairs + Rows<kThreads>::kTile - 1) / Rows<kThreads>::kTile;
        group = 1;
        while (64 * group * group < tiles) group *= 2;
        groups = (tiles + group - 1) / group;
    }
};

// Whole workgroup: f(bucket, group, the table's row of its first group) for every group that workgroup `block` of kBigBlocks takes.
// s_item: kThreads + 1 words of LDS that f leaves alone.
template <int kThreads, typename F>
__device__ __forceinline__ void big_groups(const int32_t *starts, const int32_t *big, int num_big, int block, int *s_item, int *s_wtot, F f)
{
    const int tid = threadIdx.x;
    int item0 = 0;                                          // the first group of this stretch of buckets, a thread each
    for (int e0 = 0; e0 < num_big; e0 += kThreads) {
        int groups = 0;
        if (e0 + tid < num_big) {
            const int32_t b = big[e0 + tid];
            groups = BigBucket<kThreads>(starts[b + 1] - starts[b]).groups;
        }
        const int first = row_scan<kThreads>(groups, s_wtot);
        s_item[tid] = first;
        if (tid == kThreads - 1) s_item[kThreads] = first + groups;
        __syncthreads();
        const int total = s_item[kThreads];
        for (int i = ((block - item0) % kBigBlocks + kBigBlocks) % kBigBlocks; i < total; i += kBigBlocks) {
            int lo = 0, hi = kThreads;                      // the last bucket whose groups begin at or before i
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_item[mid] <= i) lo = mid; else hi = mid;
            }
            f(big[e0 + lo], i - s_item[lo], item0 + s_item[lo]);
        }
        item0 += total;
        __syncthreads();
    }
}

// One bucket: a wave ranks its keys by row against those of its lower lanes and earlier rounds, as above, the counts of the
// workgroup's waves are added up in row order -- which gives the row pointers --, and the values leave from their places in LDS.
// kOut: the list's values are the tensors that the operators (rows) write; where they are one run of tensors -- sorted by
// operator, position e writes tensor e + shift, in any order inside an operator's row -- the rows by tensor follow from the
// rows alone and are written here, too; elsewhere kStatusPending says that they are not.
template <bool kOut, int kThreads>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6, 8)))
void k_bucket_rows(const int32_t *keys, const int32_t *vals, const int32_t *starts, int32_t buckets, int row_bits, const int32_t *big,
                   const int32_t *num_big, int32_t *big_table, EdgeList l, int32_t *status)
{
    using R = Rows<kThreads>;
    __shared__ int32_t s_val[R::kTile];
    __shared__ uint16_t s_row[kOut ? R::kTile : 1];
    __shared__ uint32_t s_count[R::kWaves][R::kRows / 2];
    __shared__ uint32_t s_seen[kOut ? R::kTile / 32 : 1];
    __shared__ int s_wtot[R::kWaves];
    if (status[kStatusNoRows]) return;                      // (a key that is no row: the starts need not ascend)
    const int lane = lane_id(), wave = threadIdx.x >> 6, tid = threadIdx.x;
    const int row_mask = (1 << row_bits) - 1;
    int *s_base = s_val;                                    // of a bucket of several tiles (no value is kept in LDS then)
    if (blockIdx.x >= (unsigned)buckets) {                  // the rows of big buckets are counted by groups of tiles
        static_assert(R::kTile >= 3 * kThreads + 1, "counts, groups of buckets");
        big_groups<kThreads>(starts, big, *num_big, (int)(blockIdx.x - buckets), s_base + 2 * kThreads, s_wtot,
                             [&](int32_t b, int group, int table0) {
            const int32_t lo = starts[b], end = starts[b + 1];
            const int32_t most = BigBucket<kThreads>(end - lo).group * R::kTile, at = lo + group * most;
            s_base[2 * tid] = s_base[2 * tid + 1] = 0;
            __syncthreads();
            count_rows<kThreads>(keys + at, min(most, end - at), b << row_bits, row_mask, s_base);
            reinterpret_cast<int2 *>(big_table + (int64_t)(table0 + group) * R::kRows)[tid] = make_int2(s_base[2 * tid], s_base[2 * tid + 1]);
        });
        return;
    }
    const int32_t b = (int32_t)blockIdx.x;
    const bool last_bucket = b == buckets - 1;
    const int32_t lo = starts[b], n = starts[b + 1] - lo;
    const int32_t row0 = b << row_bits;
    const int rows = min(1 << row_bits, l.num_ops - row0);
    const int32_t nnz = (int32_t)l.nnz, shift = l.num_tensors - nnz;
    // (once some workgroup has found that the rows by tensor are not to be had here, the others write the rows by operator alone)
    const bool together = kOut && shift >= 0 && load_coherent(&status[kStatusPending]) == 0;
    int32_t *const rowptr = l.row + row0;
    keys += lo;
    vals += lo;
    auto write_rowptr = [&](int first, int second) {
        if (2 * tid < rows) rowptr[2 * tid] = first;
        if (2 * tid + 1 < rows) rowptr[2 * tid + 1] = second;
        if (last_bucket && tid == 0) rowptr[rows] = nnz;
    };
    const bool several = n > R::kTile;                      // tiles, one after the other, every row's share behind the last tile's
    if (several) {
        if (kOut && tid == 0) store_coherent(&status[kStatusPending], 1);
        if (n > kSerialTiles * R::kTile) return;            // (k_big_rows)
        s_base[2 * tid] = s_base[2 * tid + 1] = 0;
        __syncthreads();
        count_rows<kThreads>(keys, n, row0, row_mask, s_base);
        const int v0 = s_base[2 * tid], v1 = s_base[2 * tid + 1];
        const int first = lo + row_scan<kThreads>(v0 + v1, s_wtot);
        write_rowptr(first, first + v0);
        s_base[2 * tid] = first;
        s_base[2 * tid + 1] = first + v0;
    } else if (together) {
        for (int i = tid; i < R::kTile / 32; i += kThreads) s_seen[i] = 0;
        // tensors before the run have no producer
        for (int64_t t = (int64_t)b * kThreads + tid; t < shift; t += (int64_t)buckets * kThreads) {
            l.prod_row[t] = 0;
        }
        if (last_bucket && tid == 0) l.prod_row[l.num_tensors] = nnz;
    }
    int begin = 0, length0 = 0, length1 = 0;                // of this thread's two rows, in the tile
    bool bad = false;                                       // (a list without tensors has no edges)
    const uint16_t *const mine = reinterpret_cast<const uint16_t *>(s_count[wave]);
    for (int32_t t0 = 0; t0 == 0 || t0 < n; t0 += R::kTile) {
        const int m = min((int32_t)R::kTile, n - t0);
        TilePairs p;
        rank_tile<kThreads>(keys + t0, vals + t0, m, row0, row_mask, l.num_tensors, s_count, p, bad);
        place_rows<kThreads>(s_count, length0, length1, [&](int v0, int v1) -> uint32_t {
            if (several) return 0;
            begin = row_scan<kThreads>(v0 + v1, s_wtot);
            write_rowptr(lo + begin, lo + begin + v0);
            return (uint32_t)begin | (uint32_t)(begin + v0) << 16;
        });
#pragma unroll
        for (int r = 0; r < kRowRounds; ++r) {
            if (r >= p.rounds) break;
            if (p.first + r * kWave >= m) continue;
            const int at = mine[p.row[r]] + p.rank[r];
            if (several) {
                l.idx[s_base[p.row[r]] + at] = p.val[r];
            } else {
                s_val[at] = p.val[r];
                if (kOut) s_row[at] = (uint16_t)p.row[r];
            }
        }
        __syncthreads();
        if (several) {
            s_base[2 * tid] += length0;
            s_base[2 * tid + 1] += length1;
            __syncthreads();
        }
    }
    if (ballot64(bad) != 0 && lane == 0) atomicOr(status, kErrIdRange);
    if (several) return;
    bool elsewhere = kOut && !together, scattered = false;
    for (int i = tid; i < n; i += kThreads) {
        const int32_t v = s_val[i], e = lo + i;
        l.idx[e] = v;
        if (kOut && !elsewhere) {
            const int row = s_row[i];
            const int64_t j = (int64_t)v - shift - lo;                      // the place of this tensor, in one run
            if (j < 0 || j >= n || s_row[j] != row) elsewhere = true;
            else if (atomicOr(&s_seen[j >> 5], 1u << (j & 31)) >> (j & 31) & 1) elsewhere = true;       // a second time
            scattered |= j != i;
            l.prod_idx[e] = row0 + row;
            l.prod_row[e + shift] = e;
        }
    }
    if (kOut) {
        if (ballot64(scattered) != 0 && lane == 0 && load_coherent(&status[kStatusScattered]) == 0)
            store_coherent(&status[kStatusScattered], 1);
        if (ballot64(elsewhere) != 0 && lane == 0 && load_coherent(&status[kStatusPending]) == 0)
            store_coherent(&status[kStatusPending], 1);
    }
}

// Big buckets, a workgroup per group of tiles: the counts of the bucket's groups give its rows and where this one's share of each begins.
template <int kThreads>
__global__ __launch_bounds__(kThreads)
void k_big_rows(const int32_t *keys, const int32_t *vals, const int32_t *starts, int32_t buckets, int row_bits, const int32_t *big,
                const int32_t *num_big, const int32_t *big_table, EdgeList l, int32_t *status)
{
    using R = Rows<kThreads>;
    __shared__ uint32_t s_count[R::kWaves][R::kRows / 2];
    __shared__ int s_base[R::kRows], s_item[kThreads + 1];
    __shared__ int s_wtot[R::kWaves];
    const int found = *num_big;
    if (found == 0 || status[kStatusNoRows]) return;
    const int wave = threadIdx.x >> 6, tid = threadIdx.x;
    const uint16_t *const mine = reinterpret_cast<const uint16_t *>(s_count[wave]);
    bool bad = false;
    big_groups<kThreads>(starts, big, found, (int)blockIdx.x, s_item, s_wtot, [&](int32_t b, int group, int table0) {
        const int32_t lo = starts[b], end = starts[b + 1];
        const BigBucket<kThreads> k(end - lo);
        const int32_t row0 = b << row_bits;
        const int rows = min(1 << row_bits, l.num_ops - row0);
        int all0 = 0, all1 = 0, before0 = 0, before1 = 0;   // of this thread's two rows: in the bucket, in earlier groups
        const int2 *table = reinterpret_cast<const int2 *>(big_table + (int64_t)table0 * R::kRows) + tid;
#pragma unroll 8
        for (int q = 0; q < k.groups; ++q) {
            const int2 c = table[(int64_t)q * (R::kRows / 2)];
            all0 += c.x;
            all1 += c.y;
            before0 += q < group ? c.x : 0;
            before1 += q < group ? c.y : 0;
        }
        const int first = lo + row_scan<kThreads>(all0 + all1, s_wtot);
        if (group == 0) {
            if (2 * tid < rows) l.row[row0 + 2 * tid] = first;
            if (2 * tid + 1 < rows) l.row[row0 + 2 * tid + 1] = first + all0;
            if (b == buckets - 1 && tid == 0) l.row[l.num_ops] = (int32_t)l.nnz;
        }
        s_base[2 * tid] = first + before0;
        s_base[2 * tid + 1] = first + all0 + before1;
        for (int t = group * k.group; t < min((group + 1) * k.group, k.tiles); ++t) {
            const int32_t at = lo + t * R::kTile;
            const int m = min((int32_t)R::kTile, end - at);
            TilePairs p;
            rank_tile<kThreads>(keys + at, vals + at, m, row0, (1 << row_bits) - 1, l.num_tensors, s_count, p, bad);
            int v0, v1;
            place_rows<kThreads>(s_count, v0, v1, [](int, int) -> uint32_t { return 0; });
#pragma unroll
            for (int r = 0; r < kRowRounds; ++r) {
                if (r >= p.rounds) break;
                if (p.first + r * kWave < m) l.idx[s_base[p.row[r]] + mine[p.row[r]] + p.rank[r]] = p.val[r];
            }
            __syncthreads();
            s_base[2 * tid] += v0;
            s_base[2 * tid + 1] += v1;
        }
    });
    if (ballot64(bad) != 0 && lane_id() == 0) atomicOr(status, kErrIdRange);
}

// Buckets are taken where they save a pass over memory: as many rows to a bucket as fill three quarters of a tile on average, and
// the larger tile (512 threads, ten bits) only where that takes a pass less than the smaller one: it holds a CU to three workgroups.
// Few rows with hundreds of pairs each (key bits that one pass sorts anyway) are sorted as a whole.
RowPlan plan_rows(int64_t nnz, int64_t rows, int key_bits)
{
    RowPlan p{};
    if (nnz < 1 || rows < 1) return p;
    const double mean = (double)nnz / (double)rows;
    // rows per bucket, at most, for it to fit into a tile on average
    auto fit = [&](int tile, int most_bits) {
        int bits = most_bits < key_bits ? most_bits : key_bits;
        while (bits > 0 && mean * (double)(1 << bits) * 100 > (double)(kRowFillPercent * tile)) --bits;
        return bits;
    };
    const int small = fit(Rows<256>::kTile, Rows<256>::kBits), large = fit(Rows<512>::kTile, Rows<512>::kBits);
    auto passes = [&](int bits) { return sort_pass_count(key_bits - bits); };
    p.threads = passes(small) <= passes(large) ? 256 : 512;
    p.row_bits = p.threads == 256 ? small : large;
    p.passes = passes(p.row_bits);
    p.pass_bits = p.passes ? (key_bits - p.row_bits + p.passes - 1) / p.passes : 0;
    if (p.pass_bits < 6) p.pass_bits = 6;
    p.buckets = (rows + ((int64_t)1 << p.row_bits) - 1) >> p.row_bits;
    p.use = p.row_bits > 0 && p.passes < sort_pass_count(key_bits) && (size_t)(p.buckets + 1) * 4 <= sort_tmp(nullptr, nnz).table_bytes;
    return p;
}

template <int kThreads>
static hipError_t bucket_rows(const RowPlan &p, const int32_t *keys, const int32_t *vals, int32_t *big_table, const EdgeList &l, bool producers,
                              int32_t *num_big, int32_t *status, const SortTmp &t, hipStream_t s)
{
    const int32_t buckets = (int32_t)p.buckets, most = kSerialTiles * Rows<kThreads>::kTile;
    int32_t *starts = t.table, *big = t.totals;             // (the passes are done with them)
    hipLaunchKernelGGL(k_bucket_starts, dim3((unsigned)(buckets / (256 / kProbes) + 1)), dim3(256), 0, s, keys, (int32_t)l.nnz, p.row_bits,
                       buckets, most, starts, big, (int32_t)(l.nnz / most) + 1, num_big, status);
    // (a short list has no big bucket)
    const bool may_be_big = l.nnz > most;
    const dim3 grid((unsigned)(buckets + (may_be_big ? kBigBlocks : 0)));
    if (producers)
        hipLaunchKernelGGL((k_bucket_rows<true, kThreads>), grid, dim3(kThreads), 0, s, keys, vals, starts, buckets, p.row_bits, big, num_big,
                           big_table, l, status);
    else
        hipLaunchKernelGGL((k_bucket_rows<false, kThreads>), grid, dim3(kThreads), 0, s, keys, vals, starts, buckets, p.row_bits, big, num_big,
                           big_table, l, status);
    if (may_be_big)
        hipLaunchKernelGGL(k_big_rows<kThreads>, dim3(kBigBlocks), dim3(kThreads), 0, s, keys, vals, starts, buckets, p.row_bits, big, num_big,
                           big_table, l, status);
    return hipGetLastError();
}

hipError_t launch_bucket_rows(const RowPlan &p, const EdgeList &l, bool producers, int32_t *num_big, int32_t *status, void *tmp, hipStream_t s)
{
    const SortTmp t = sort_tmp(tmp, l.nnz);
    const int32_t *keys = l.op, *vals = l.tensor;
    if (p.passes == 0) {
        const hipError_t e = launch_check_ids(l, status, s);
        if (e != hipSuccess) return e;
    } else {
        const hipError_t e = p.pass_bits == 6 ? sort_passes<6>(keys, vals, nullptr, nullptr, l.nnz, p.row_bits, p.passes, t, s, l.num_ops, status)
                           : p.pass_bits == 7 ? sort_passes<7>(keys, vals, nullptr, nullptr, l.nnz, p.row_bits, p.passes, t, s, l.num_ops, status)
                           : p.pass_bits == 8 ? sort_passes<8>(keys, vals, nullptr, nullptr, l.nnz, p.row_bits, p.passes, t, s, l.num_ops, status)
                                              : sort_passes<9>(keys, vals, nullptr, nullptr, l.nnz, p.row_bits, p.passes, t, s, l.num_ops, status);
        if (e != hipSuccess) return e;
        keys = t.keys[(p.passes - 1) & 1];
        vals = t.vals[(p.passes - 1) & 1];
    }
    // counts of the big buckets' groups of tiles, a byte per pair of a tile each: in the buffer that the last pass read
    int32_t *big_table = t.keys[p.passes & 1];
    return p.threads == 256 ? bucket_rows<256>(p, keys, vals, big_table, l, producers, num_big, status, t, s)
                            : bucket_rows<512>(p, keys, vals, big_table, l, producers, num_big, status, t, s);
}

}  // namespace dgn
