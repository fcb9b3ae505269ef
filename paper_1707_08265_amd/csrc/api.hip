// C ABI of libdgn: argument checking, workspace layout and kernel sequencing (declared in dgn.h).
// Host code only decides *which* kernels run and where their buffers live; every step of the path
// itself (adjacency build, seeding, traversal, removal rule, compaction) is a device kernel.
#include <math.h>
#include <new>
#include <string.h>

#include "common.h"

#include <atomic>

using namespace dgn;

namespace {

thread_local int t_last_hip = 0;

inline int hip_fail(hipError_t e)
{
    t_last_hip = (int)e;
    return DGN_ERR_HIP;
}
#define DGN_HIP(expr)                                   \
    do {                                                \
        hipError_t e__ = (expr);                        \
        if (e__ != hipSuccess) return hip_fail(e__);    \
    } while (0)

constexpr int64_t kMaxCount = 2147483646;   // counts must stay below 2^31 - 1
constexpr int kLevelBlocksPerCU = 5;   // workgroups of a wide level per compute unit
// Frontiers up to this size are walked by one workgroup (one round of its threads); in graphs that read nearby only smaller
// ones.  Those are deep (an unrolled RNN: a level per 30 operators of a step), and a level of several hundred entries takes
// one workgroup 7 us where the 32 hops of a wide launch take 3 us each: 900 000 operators, 33 targets 262 -> 193 us, two million
// 220 -> 158.  A power-law graph is through after a few levels (300 000 operators, one target: 137 us, the other way 190).
// A prune that starts with the one workgroup lets it have frontiers up to kNarrowCap in any graph: often it is through then,
// and where nothing is known the other way is 48 wide launches ahead (300 000 operators, 64 sets, first prune 145 us, 252).
constexpr int kNarrowCap = 1024, kNarrowCapNear = 320;
constexpr int kNarrowLevels = 12;           // done by the one workgroup in so few levels, a prune is left to it (100 000 operators
                                            // in 12 levels 127 us, wide 138; 36 000 in 13 144, wide 111)
constexpr int kWidePerGroup = 12;           // wide level launches between two single-workgroup launches
// Groups in the batches of a graph not known yet (one state read-back per batch): one or two in the first (see first_groups), then one --
// most graphs that the first was too short for need little more --, two, four, and this.  (Twice as many as before each time, from the
// first batch on: the same within 2 % for 60 first prunes of twelve graphs.)
constexpr int kWideGroups = 6;
constexpr int64_t kOneGroupOps = (int64_t)1 << 16, kOneGroupFlatOps = (int64_t)1 << 19;
constexpr int kMaxBatch = 512;              // launches enqueued between two state read-backs, at most
constexpr int kTailLevels = 1;              // wide launches enqueued beyond the layout the previous prune needed ...
constexpr int kExactStreak = 3;             // ... until that layout has fitted exactly this many prunes in a row
constexpr int kBackwardMaxBatch = 60;       // forward passes of the backward prune between two read-backs, at most
constexpr int kSweepMinGraphs = 64;         // packed batches with at least this many graphs ...
constexpr int64_t kSweepMaxGraphOps = 1 << 18;   // ... none larger than this use the per-graph sweep
constexpr u64 kRecycleMagic = 0x44474e5f52435943ull;   // "DGN_RCYC"
constexpr u64 kRingMagic = 0x44474e5f52494e47ull;      // "DGN_RING": a result of the ring sweep (bitmap, no log)
constexpr u64 kBandMagic = 0x44474e5f42414e44ull;      // "DGN_BAND": a result of the sweep by layers
constexpr int64_t kRingSeedWords = 2048;               // targets of a graph that the ring sweep keeps in LDS, at most
// Which graphs may take the ring sweep (see ring_waves):
constexpr int64_t kRingMaxOps = (int64_t)1 << 17;      // single graphs, or fewer than the per-graph sweep starts at: at most this
constexpr int64_t kRingShortOps = 16384;               // size, and, times the words of sets, up to this
constexpr int64_t kRingAboutOps = 4096;                // ... to this when operators read from all over the graph,
constexpr int64_t kRingThinOps = 20480;                // ... to this when no input lies further back
constexpr int kRingThinDist = 96;                      // than this, or to any size once a prune has taken
constexpr int kRingLongLevel = 256;                    // more than a level per so many operators of the largest graph
// (graphs of a larger batch: kRingMaxGraphOps)
// When such a graph is swept in segments, and how long they are (see ring_segments):
constexpr double kRingWordUs = 0.9, kRingSegmentsUs = 6.5, kRingSegmentOpUs = 2.5e-5;
constexpr double kRingManyWordUs = 0.71, kRingManySegWordUs = 1.06, kRingManyUs = 2.0, kRingManyOpUs = 0.9e-5, kRingManyTargetUs = 0.007;
constexpr double kRingFromMUs = 15.0, kRingFromMTargetUs = 0.0028;
constexpr int kRingFewWords = 16, kRingManySegs = 64, kRingSegmentsPerCu = 24, kRingFewSegmentsPerCu = 2;
// Which single graphs are swept by layers (see band_sweep.hip), of those that the ring sweep leaves: they read the last eighth of the
// graph mostly, and no more than one operator in 25 what was written just before (layers of 40: one in 100, chains with a window of
// 64: one in 10).  Whole prunes, level by level / swept, 64 sets of up to 8: 24 layers of 700 161 / 82 us, 60 x 300 173 / 86, 200 x 90
// 170 / 119, 500 x 400 370 / 216, 1 000 x 40 376 / 284, 1 000 x 800 817 / 661; first prunes of them 300 to 800 / 92 to 674.  With a
// single set of 4: 24 x 700 96 / 64, 100 x 600 159 / 111, 500 x 400 255 / 209, but 300 x 667 206 / 226, 300 x 800 210 / 232, 500 x 700 267 /
// 337 and 1 000 x 600 471 / 591, so up to four sets on more than 200 000 operators are left to the levels, or on more than 300 000 where
// there are some 600 layers and more, which fit a step each then (600 x 450 317 / 245, 1 000 x 210 424 / 291, 1 000 x 300 407 / 324, but 700 x
// 560 362 / 415).  At four sets the two ways meet (300 x 667 234 / 227, 500 x 700 332 / 339, 1 000 x 600 567 / 594), from five on the sweep is
// the faster one or takes the same time (255 / 228, 345 / 340, 586 / 595; eight: 265 / 230, 370 / 340, 617 / 597).
//   More than kBandMaxTargets targets go by way of M, and a step of the sweep takes half as long again; the levels take no longer than
// with few.  Up to 50 000 operators and 8 000 for every set the sweep is the faster one or takes the same time (100 x 500 128 / 112; 1 000 x 40
// 350 / 355; four sets on 100 x 600 150 / 134, eight on 300 x 200 183 / 167, but on 200 x 600 190 / 212 and 450 x 700 304 / 421; five on 1 000 x 600
// 523 / 787), with sixteen sets and more up to 300 000 (32 sets, 500 x 400 328 / 284, 1 000 x 300 500 / 425; 64 sets 345 / 284, 535 / 425,
// but 1 000 x 600 680 / 788, 1 000 x 800 822 / 872; sixteen are the limit: 500 x 400 308 / 275, 300 x 667 260 / 300), and with five and more
// where there are some 700 layers and more (eight sets on 1 000 x 250 449 / 406).
constexpr int kBandSoonShare = 25;
constexpr int64_t kBandFewSets = 4, kBandFewSetsOps = 200000, kBandFewSetsDeepOps = 300000, kBandLastWordDeepOps = 400000;
constexpr int64_t kBandFromMOps = 50000, kBandFromMSetOps = 8000, kBandFromMManySets = 16, kBandFromMMaxOps = 300000;
constexpr int kSmallLevel = 16384;           // levels expanding fewer entries than this decay the threshold faster
constexpr int kDefaultDeferPercent = 74;
constexpr int kDefaultStartShift = 1;       // deferral threshold starts at P >> 1 ...
constexpr int kDefaultFloorShift = 10;      // ... and stops (drops to 0) below P >> 10 or, in large graphs,
constexpr int kDefaultFloorPerRoot = 2;     // below 2 sqrt(P); earlier, at
constexpr int kNearFloorShift = 3;          // P >> 3, in graphs that read nearby, but in many hundred layers not for
constexpr int kFewSets = 8;                 // so few sets and
constexpr double kFewSetsOps = 450000;      // so few operators times the root of their number; and where there are many targets,
constexpr int64_t kLayeredTargets = 256;    // in graphs of a few dozen layers or more
constexpr int64_t kDeepTargets = 512;       // in deep graphs no larger than
constexpr int64_t kDeepOps = (int64_t)1 << 22;

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// carve consecutive 256-byte aligned regions out of one buffer
struct Carver {
    char *base;
    size_t off = 0;
    explicit Carver(void *p) : base(static_cast<char *>(p)) {}
    template <typename T> T *take(size_t count)
    {
        T *r = base ? reinterpret_cast<T *>(base + off) : nullptr;
        off += align256(count * sizeof(T));
        return r;
    }
};

inline int key_bits_for(int64_t n)
{
    int b = 1;
    while (b < 31 && ((int64_t)1 << b) < n) ++b;
    return b;
}

int check_sizes(int64_t P, int64_t T, int64_t Ein, int64_t Eout, int32_t G, const int64_t *op_off,
                const int64_t *t_off)
{
    if (P < 0 || T < 0 || Ein < 0 || Eout < 0 || G < 1) return DGN_ERR_INVALID_ARG;
    if (P > kMaxCount || T > kMaxCount || Ein > kMaxCount || Eout > kMaxCount) return DGN_ERR_TOO_LARGE;
    if (G > 1) {
        if (!op_off || !t_off) return DGN_ERR_NULL_PTR;
        if (op_off[0] != 0 || t_off[0] != 0 || op_off[G] != P || t_off[G] != T) return DGN_ERR_INVALID_ARG;
        for (int32_t g = 0; g < G; ++g)
            if (op_off[g + 1] < op_off[g] || t_off[g + 1] < t_off[g]) return DGN_ERR_INVALID_ARG;
    }
    return DGN_OK;
}

// Operators of the largest graph.
int64_t largest_graph(int64_t P, int32_t G, const int64_t *op_off)
{
    if (G == 1) return P;
    int64_t most = 0;
    for (int32_t i = 0; i < G; ++i) most = op_off[i + 1] - op_off[i] > most ? op_off[i + 1] - op_off[i] : most;
    return most;
}

// Batches that are swept have no records: what goes operator by operator over such a batch takes its rows, and from 4 instead of 16 bytes per
// operator which tensors it writes.  (4 096 graphs of 20 000: records and check 741 us with records, 600 so.)  A batch with a larger graph than
// that goes level by level, and has them (64 graphs of 300 000, 64 sets: prune 36.05 ms with records, 36.35 without, build 483 us, 449).  Levels of a swept batch,
// where an option asks for them or its operators are in no topological order, do without (4 096 graphs of 20 000: 52.6 ms / 54.4, the
// sweep takes 1.1; 64 in reverse order 1.89 / 1.94, 256 3.10 / 3.10 and their build 797 us / 785).
bool is_swept(int32_t G, int64_t max_graph_ops) { return G >= kSweepMinGraphs && max_graph_ops <= kSweepMaxGraphOps; }
static_assert(kRingMaxGraphOps <= kSweepMaxGraphOps, "what takes either sweep has no records");

struct GraphLayout {
    int32_t *in_rowptr, *in_idx, *out_rowptr, *out_idx, *prod_rowptr, *prod_idx;
    Quad *orec;             // NULL: a batch that is swept, which has ...
    int32_t *ofirst;        // ... these
    int32_t *prod1;
    int64_t *op_off, *t_off;
    int64_t max_graph_ops;
    size_t bytes;
};

GraphLayout graph_layout(void *mem, int64_t P, int64_t T, int64_t Ein, int64_t Eout, int32_t G, const int64_t *op_off, bool own_op_csr)
{
    Carver c(mem);
    GraphLayout L{};
    if (own_op_csr) {
        L.in_rowptr = c.take<int32_t>(P + 1);
        L.in_idx = c.take<int32_t>(Ein);
        L.out_rowptr = c.take<int32_t>(P + 1);
        L.out_idx = c.take<int32_t>(Eout);
    }
    L.prod_rowptr = c.take<int32_t>(T + 1);
    L.prod_idx = c.take<int32_t>(Eout);
    L.max_graph_ops = largest_graph(P, G, op_off);
    if (is_swept(G, L.max_graph_ops)) L.ofirst = c.take<int32_t>(P);
    else L.orec = c.take<Quad>(P);
    L.prod1 = c.take<int32_t>(T);
    if (G > 1) {
        L.op_off = c.take<int64_t>(G + 1);
        L.t_off = c.take<int64_t>(G + 1);
    }
    L.bytes = c.off > 0 ? c.off : 256;
    return L;
}

struct BuildScratch {
    int32_t *status;        // [kStatusEnd]; status[0] = error bits
    int32_t *sorted_ops;    // [Eout] operator id of every entry of out_idx
    int32_t *sorted_keys;   // [max(Ein, Eout)] keys of a sort in row order, for the row pointers
    void *sort_tmp;
    size_t bytes;
};

BuildScratch build_scratch(void *mem, int64_t Ein, int64_t Eout)
{
    Carver c(mem);
    BuildScratch S{};
    S.status = c.take<int32_t>(kStatusEnd);
    S.sorted_ops = c.take<int32_t>(Eout);
    const int64_t emax = Ein > Eout ? Ein : Eout;
    S.sorted_keys = c.take<int32_t>(emax);
    S.sort_tmp = c.take<char>(sort_tmp_bytes(emax));
    S.bytes = c.off;
    return S;
}

struct PruneScratch {
    TravState *state;
    TravCounters *ctr;
    int32_t *q0, *q1;       // frontier queues: qg.S segments of qg.seg_cap tensor ids each
    QueueGeom qg;
    uint8_t *DB;            // deferred-operator markers, one byte per operator
    uint8_t *flagbuf;       // keep flags (a byte per operator) when the caller's op_flag cannot take them
    u64 *opbits;
    int32_t *block_counts;
    Quad *trace;            // per-level trace records (profiling only)
    int64_t *pq_part;       // replicated per-set counters (few graphs only), NULL otherwise
    int pq_replicas;
    size_t pq_part_bytes;
    size_t db_bytes, opbits_bytes;
    RecycleHeader *hdr;     // says which buffers hold the result of the last prune that kept a complete log
    ColourLog log;          // tensors that prune coloured
    u64 *ring_bits;         // ring sweep: a bit per operator, running counts per word, a record per graph
    int32_t *ring_cum;
    Quad *ring_graphs;
    const char *end;        // of the buffer
    size_t bytes;
};

// Where the ring sweep keeps its flag bytes: the caller's op_flag when the traversal could clear that in whole 8-byte words
// (a later call recycles either's result), else the scratch array, if there is one.
uint8_t *ring_flags(const PruneScratch &S, uint8_t *op_flag, int64_t P)
{
    const bool whole = op_flag && ((uintptr_t)op_flag & 7) == 0 && P % 8 == 0;
    return whole || !S.flagbuf ? op_flag : S.flagbuf;
}

// Segments: enough of them that no push counter sees more than a few hundred waves per level, few
// enough that tiny graphs do not pay for empty segments.  Total capacity 2T + slack: a level can hold
// more than T entries because the frontier is not deduplicated (beyond that, the overflow path runs).
QueueGeom queue_geometry(int64_t T, int64_t max_entries)
{
    int S = 1;
    while (S < kMaxSeg && (int64_t)S * 16384 < T) S *= 2;
    int64_t total = 2 * T + 1024;
    if (max_entries > 0 && max_entries < total) total = max_entries;
    int64_t seg = (total + S - 1) / S;
    if (seg < 1) seg = 1;
    return QueueGeom{S, (int32_t)seg};
}

// whole_queues: room for full queues also where max_entries makes them smaller
PruneScratch prune_scratch(void *mem, int64_t P, int64_t T, int32_t G, int64_t max_entries, bool whole_queues = false)
{
    Carver c(mem);
    PruneScratch S{};
    // What one prune leaves for the next comes first, where no option moves it.  Log of coloured tensors: a
    // quarter of T in all.  Recycling only pays while a prune colours a small part of the graph; one that
    // overflows the log makes the next prune clear everything, as if there were no log.
    S.hdr = c.take<RecycleHeader>(4);
    S.log.cnt = c.take<SegCounter>(kMaxSeg);
    int64_t lcap = T / (4 * kMaxSeg);
    if (lcap < 4096) lcap = 4096;
    S.log.seg_cap = (int32_t)lcap;
    S.log.entries = c.take<int32_t>((size_t)kMaxSeg * (size_t)lcap);
    if (G > 1 || P <= kRingMaxOps) {
        const size_t words = (size_t)ring_bit_words(P, G);
        S.ring_bits = c.take<u64>(words);
        S.ring_cum = c.take<int32_t>(words);
        S.ring_graphs = c.take<Quad>((size_t)G + 1);
    }
    S.state = c.take<TravState>(2);
    S.ctr = c.take<TravCounters>(1);
    S.qg = queue_geometry(T, max_entries);
    const QueueGeom room = whole_queues ? queue_geometry(T, 0) : S.qg;
    const size_t qn = (size_t)room.S * (size_t)room.seg_cap;
    S.q0 = c.take<int32_t>(qn);
    S.q1 = c.take<int32_t>(qn);
    const size_t obw = (size_t)((P + 63) / 64);
    S.DB = c.take<uint8_t>(obw * 64);         // a whole number of 64-operator words, so chunk loads stay inside
    S.db_bytes = obw * 64;
    S.flagbuf = c.take<uint8_t>(obw * 64);
    S.opbits = c.take<u64>(obw);
    S.opbits_bytes = obw * 8;
    S.block_counts = c.take<int32_t>((P + kCompactTile - 1) / kCompactTile + 1);
    S.trace = c.take<Quad>(kTraceLevels);
    // with fewer than 64 graphs the 64*G per-set counters would be hot words: replicate them
    S.pq_replicas = 1;
    while (S.pq_replicas * 2 * (int64_t)G <= 64) S.pq_replicas *= 2;
    S.pq_part_bytes = S.pq_replicas > 1 ? sizeof(int64_t) * 64 * (size_t)G * S.pq_replicas * kPqStride : 0;
    S.pq_part = c.take<int64_t>(S.pq_part_bytes / sizeof(int64_t));
    if (S.pq_replicas == 1) S.pq_part = nullptr;
    S.bytes = c.off;
    S.end = mem ? static_cast<const char *>(mem) + S.bytes : nullptr;
    return S;
}

// Lays out everything behind the log again for the ring sweep of several words of 64 sets at once, `words` of them or as many
// as have room (returned; below two nothing is changed).  Flag bytes have no place in that layout: nothing is recycled, so
// nobody reads them back.
int64_t words_scratch(PruneScratch &S, void *scratch, int64_t P, int64_t words)
{
    const size_t per = (size_t)ring_bit_words(P, 1);
    char *room = reinterpret_cast<char *>(S.ring_bits);
    const size_t bytes = S.bytes - (size_t)(room - static_cast<char *>(scratch));
    int64_t at_once = (int64_t)((bytes - 3 * 256) / (per * (sizeof(u64) + sizeof(int32_t)) + sizeof(Quad)));
    if (at_once > words) at_once = words;
    if (at_once < 2) return 1;
    Carver c(room);
    S.ring_bits = c.take<u64>(per * (size_t)at_once);
    S.ring_cum = c.take<int32_t>(per * (size_t)at_once);
    S.ring_graphs = c.take<Quad>((size_t)at_once);
    S.flagbuf = nullptr;
    return at_once;
}

// What the segments of a ring sweep may use: what lies behind one word's records, up to the flag bytes, or behind those of several, up
// to the end (flagbuf == NULL: laid out by words_scratch).
struct Room { char *at; size_t bytes; };
Room segments_room(const PruneScratch &S, int64_t words)
{
    char *at = S.flagbuf ? reinterpret_cast<char *>(S.q0) : reinterpret_cast<char *>(S.ring_graphs) + align256((size_t)words * sizeof(Quad));
    const char *end = S.flagbuf ? reinterpret_cast<const char *>(S.flagbuf) : S.end;
    return {at, at < end ? (size_t)(end - at) : 0};
}

// One small pinned buffer per host thread for status read-backs (never freed: a few hundred bytes).
int pinned_buffer(void **out)
{
    thread_local void *buf = nullptr;
    if (!buf) DGN_HIP(hipHostMalloc(&buf, 256, hipHostMallocDefault));
    *out = buf;
    return DGN_OK;
}

// Events for options->profile, created once per host thread.
int profile_events(hipEvent_t **out)
{
    thread_local hipEvent_t ev[8];
    thread_local bool ready = false;
    if (!ready) {
        for (int i = 0; i < 8; ++i) DGN_HIP(hipEventCreate(&ev[i]));
        ready = true;
    }
    *out = ev;
    return DGN_OK;
}

int error_bits_to_code(int32_t bits)
{
    if (bits & kErrCsr) return DGN_ERR_BAD_CSR;
    if (bits & (kErrIdRange | kErrCrossGraph)) return DGN_ERR_ID_OUT_OF_RANGE;
    if (bits & kErrTopo) return DGN_ERR_NOT_TOPOLOGICAL;
    return DGN_OK;
}

int check_options(const dgn_options *o)
{
    if (!o) return DGN_OK;
    if (o->traversal < 0 || o->traversal > 2) return DGN_ERR_INVALID_ARG;
    if (o->defer_percent < 0 || o->defer_percent > 100) return DGN_ERR_INVALID_ARG;
    if (o->max_queue_entries < 0) return DGN_ERR_INVALID_ARG;
    if (o->recycle < 0 || o->recycle > 1) return DGN_ERR_INVALID_ARG;
    if (o->profile < 0 || o->profile > 2) return DGN_ERR_INVALID_ARG;
    if (o->defer_start_shift < 0 || o->defer_start_shift > 30) return DGN_ERR_INVALID_ARG;
    if (o->defer_floor_shift < 0 || o->defer_floor_shift > 30) return DGN_ERR_INVALID_ARG;
    return DGN_OK;
}

}  // namespace

// How far back half of the operators read at most (sampled, single graphs with their outputs in one run of tensors)
enum class Reach { unknown, layers /* a 32nd of the graph */, near /* a 192nd */, nearer /* a 640th */, deep /* a 2 048th */ };

struct dgn_graph {
    GraphView v;
    int64_t P, T, Ein, Eout;
    int32_t G;
    int num_cus;
    bool topological;       // operator ids verified to be a topological order at build time
    bool multi_producer;    // some tensor is written by more than one operator
    int64_t max_graph_ops;  // largest graph of a packed batch (P for a single graph)
    bool ring;              // the ring sweep can take these graphs: see ring_sweep.hip for the three numbers
    int ring_low, ring_dist, ring_span64, ring_reach;
    Reach reach;            // how far back the operators of a single graph read (see the schedule in prune_impl)
    Meet meet;              // what many operators read at the same time (see the in-place pass)
    bool reads_about;       // half of the operators (of all graphs) read further back than an eighth of their graph, or nobody knows
    bool layers;            // a single graph, its outputs in one run of tensors, that looks like layers (see band_sweep.hip)
    uint64_t serial;        // unique per handle in this process
    // Hints only, taken from the last prune of this graph; a wrong one costs launches that return at once,
    // or a second batch, and corrects itself.  Kept apart for full prunes [0] and incremental ones [1],
    // whose traversals look nothing alike.
    //   wide_hint: wide levels were needed, so they are enqueued behind the first single-workgroup launch
    //     without waiting for its outcome;
    //   hint_runs, hint_run_len: how that prune alternated between stretches of wide levels and the
    //     single-workgroup kernel (lengths of the first stretches; 0 stretches: unknown); the launches are
    //     laid out the same way instead of in fixed groups.
    //   long_chains: a prune of this graph took so many levels that the ring sweep is the better way for it (see ring_waves)
    //   no_layers: the plan of the sweep by layers has found that the graph is not of that kind
    mutable std::atomic<int> long_chains = {};
    mutable std::atomic<int> no_layers = {};
    mutable std::atomic<int> wide_hint[2] = {};
    mutable std::atomic<int> hint_runs[2] = {};
    mutable std::atomic<int> hint_run_len[2][dgn::kMaxRuns] = {};
    //   exact_streak: prunes in a row whose traversal followed the hinted layout to the launch; after a few the
    //     spare launches at its end are dropped (a miss then costs one more batch, and brings them back)
    mutable std::atomic<int> exact_streak[2] = {};
    //   backward_passes: forward passes the last backward prune of this graph needed; the next one enqueues that many
    //     before it looks at their outcome
    mutable std::atomic<int> backward_passes = {};
};

namespace {

constexpr int kStatusWords = kStatusSoon + 1;

// The status words of a build, once everything before them is done.
int read_status(const int32_t *status, hipStream_t s, const int32_t **out)
{
    void *pin = nullptr;
    const int rc = pinned_buffer(&pin);
    if (rc) return rc;
    DGN_HIP(hipMemcpyAsync(pin, status, kStatusWords * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    DGN_HIP(hipStreamSynchronize(s));
    *out = static_cast<const int32_t *>(pin);
    return DGN_OK;
}

// Packed batches, and single graphs that the ring sweep may take, are checked in the walk that makes the records.
bool walked(const dgn_graph *h) { return h->G > 1 || h->P <= kRingMaxOps; }

// The pass over the outputs leaves out the producer words of what may be one run of tensors up to the last.  A batch's outputs hardly
// ever are: its graphs have inputs of their own.
bool may_run(const dgn_graph *h) { return h->G == 1; }

// What follows the adjacency.  The kernels find out by themselves whether there is one yet.  words: all producer words are there; none: the
// outputs are one run, or there is no adjacency yet, so that there are no records to be made.
int enqueue_records(const dgn_graph *h, const GraphLayout &L, int32_t *status, const dgn_options *options, hipStream_t s, bool words, bool none = false)
{
    int32_t *spared = may_run(h) && !words ? L.prod1 : nullptr;
    if (walked(h)) {
        DGN_HIP(launch_records_and_check(h->v, L.orec, L.ofirst, spared, status, h->num_cus, s));
    } else {
        if (none) DGN_HIP(launch_sample_reach(h->v, status, s));
        else DGN_HIP(launch_build_records(h->v, L.orec, spared, status, s));
        if (options && options->validate) DGN_HIP(launch_check_topological(h->v, status, s));
    }
    return DGN_OK;
}

// Rows by l.op of a list in no order, whose ids are checked unless they are known to be good.  big: status word.
int sort_rows(const EdgeList &l, const BuildScratch &S, bool buckets, bool good, int big, hipStream_t s)
{
    const RowPlan plan = plan_rows(l.nnz, l.num_ops, key_bits_for(l.num_ops));
    if (buckets && plan.use) {
        DGN_HIP(launch_bucket_rows(plan, l, false, S.status + big, S.status, S.sort_tmp, s));
        return DGN_OK;
    }
    if (!good) DGN_HIP(launch_check_ids(l, S.status, s));
    DGN_HIP(launch_sort_pairs(l.op, l.tensor, S.sorted_keys, l.idx, l.nnz, key_bits_for(l.num_ops), S.sort_tmp, s));
    DGN_HIP(launch_row_bounds(S.sorted_keys, l.nnz, l.num_ops, l.row, S.status, s));
    return DGN_OK;
}

// Tensor -> producer rows by a stable sort of the outputs in operator order (outputs by tensor: each tensor's producers stay
// ascending in operator id), or, if only long gaps were left out, from the list in order by tensor; then the producer words.
// buckets: by way of buckets where that is the shorter way.
int build_producers(const dgn_graph *h, const GraphLayout &L, const BuildScratch &S, const int32_t *ops_of_out,
                    const int32_t *keys, bool buckets, hipStream_t s)
{
    if (keys) {
        DGN_HIP(launch_row_bounds(keys, h->Eout, (int32_t)h->T, L.prod_rowptr, S.status, s));
    } else {
        const EdgeList list{h->v.out_idx, ops_of_out, h->Eout, (int32_t)h->T, (int32_t)h->P, L.prod_idx, L.prod_rowptr, nullptr, nullptr, nullptr, false};
        const int rc = sort_rows(list, S, buckets, true, kStatusBig + 2, s);
        if (rc) return rc;
    }
    DGN_HIP(launch_build_producers(h->v, L.prod1, S.status, s));
    return DGN_OK;
}

int copy_offsets(dgn_graph *h, const GraphLayout &L, const int64_t *op_off_host, const int64_t *t_off_host, hipStream_t s)
{
    if (h->G > 1) {
        DGN_HIP(hipMemcpyAsync(L.op_off, op_off_host, sizeof(int64_t) * (h->G + 1), hipMemcpyHostToDevice, s));
        DGN_HIP(hipMemcpyAsync(L.t_off, t_off_host, sizeof(int64_t) * (h->G + 1), hipMemcpyHostToDevice, s));
        h->v.op_off = L.op_off;
        h->v.t_off = L.t_off;
    }
    return DGN_OK;
}

// found: the status words as enqueue_records' kernels left them on an adjacency that is complete.
int finish_build(dgn_graph *h, const int64_t *op_off_host, const int64_t *t_off_host, int32_t *status, const int32_t *found,
                 const dgn_options *options, hipStream_t s, dgn_graph **out)
{
    const int32_t *ring = found + kStatusRing;
    // (32-bit byte offsets inside a graph's arrays)
    h->ring = walked(h) && h->P > 0 && h->Ein > 0 && h->Ein < (1 << 30) && h->T < (1 << 29) && ring[0] == 0;
    h->ring_low = ring[1];
    h->ring_dist = ring[2];
    h->ring_span64 = ring[3];
    h->ring_reach = found[kStatusReach];
    h->v.run_shift = found[kStatusNoRun] == 0 ? (int32_t)(h->T - h->Eout) : -1;
    h->multi_producer = found[kStatusMulti] != 0;
    auto most = [&](int word) { return found[word] * 2 > found[kStatusSampled]; };
    h->reads_about = !most(kStatusWithin8);
    if (h->G == 1)
        h->reach = most(kStatusWithin2048) ? Reach::deep : most(kStatusWithin640) ? Reach::nearer
                 : most(kStatusWithin192) ? Reach::near : most(kStatusWithin32) ? Reach::layers : Reach::unknown;
    // (operators that read what was written just before: chains, not layers)
    const bool chains = found[kStatusSoon] * kBandSoonShare > found[kStatusSampled];
    h->meet = h->G > 1 ? Meet::batch : found[kStatusSampled] == 0 ? Meet::unknown : chains ? Meet::chains : Meet::nowhere;
    h->layers = h->G == 1 && h->P > 0 && h->P <= kBandMaxOps && h->Ein > 0 && found[kStatusScattered] == 0 && h->T >= h->Eout &&
                h->T - h->Eout <= kBandMaxLow && !h->reads_about &&
                found[kStatusSoon] * kBandSoonShare <= found[kStatusSampled];
    // The topological precondition is checked when the caller asks for validation, and for packed
    // batches, whose per-graph sweep is only chosen when it holds.  (One random access per edge: not
    // worth paying on every build of a big single graph, whose traversal does not depend on it.)  Where the walk found
    // every graph's outputs in one run and no operator that reads too late, it holds.
    const bool check_topo = (options && options->validate) || h->G >= kSweepMinGraphs;
    if (check_topo && walked(h) && ring[0] != 0 && found[0] == 0) {
        FillRegion clr[1] = {{status, kStatusOrder * sizeof(int32_t)}};
        DGN_HIP(launch_clear(clr, 1, s));
        DGN_HIP(launch_check_topological(h->v, status, s));
        const int rc = read_status(status, s, &found);
        if (rc) return rc;
    }
    int32_t bits = found[0];
    h->topological = check_topo && (bits & kErrTopo) == 0;
    if (!(options && options->validate)) bits &= ~kErrTopo;
    const int rc = error_bits_to_code(bits);
    if (rc) return rc;
    for (int32_t i = 0; h->G > 1 && i < h->G; ++i)           // a graph without operators: all its tensors are inputs
        if (op_off_host[i + 1] == op_off_host[i] && t_off_host[i + 1] - t_off_host[i] > h->ring_low)
            h->ring_low = (int)(t_off_host[i + 1] - t_off_host[i]);
    static std::atomic<uint64_t> next_serial{1};
    h->serial = next_serial.fetch_add(1, std::memory_order_relaxed);
    *out = h;
    return DGN_OK;
}

// A handle with the compute units of the current device.
int new_graph(dgn_graph **out)
{
    int dev = 0, cus = 0;
    DGN_HIP(hipGetDevice(&dev));
    DGN_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    dgn_graph *h = new (std::nothrow) dgn_graph();
    if (!h) return DGN_ERR_INVALID_ARG;
    h->num_cus = cus > 0 ? cus : 256;
    *out = h;
    return DGN_OK;
}

// What is left of an adjacency when the pass over the edge lists has found (f) that they are not in order, as its status words say.
// Stable sorts, by way of buckets where that is the shorter way: edges by operator, rows keep COO order; no histogram of the rows, no
// atomics on memory.
int sort_lists(const dgn_graph *h, const EdgeList &in, const EdgeList &out, const GraphLayout &L, const BuildScratch &S,
               const int32_t (&f)[kStatusOrder], const dgn_options *options, hipStream_t s, const int32_t **found)
{
    const int64_t P = h->P, T = h->T, Eout = h->Eout;
    FillRegion clr[1] = {{S.status, 256}};
    const bool out_unsorted = f[kStatusOutUnsorted];
    bool out_gap = f[kStatusOutGap], prod_unsorted = f[kStatusProdUnsorted], prod_gap = f[kStatusProdGap];
    FillRegion order[1] = {{S.status, kStatusOrder * sizeof(int32_t)}};
    DGN_HIP(launch_clear(out_unsorted ? clr : order, 1, s));
    int rc = DGN_OK;
    if (f[kStatusInUnsorted]) {
        rc = sort_rows(in, S, true, false, kStatusBig, s);
        if (rc) return rc;
    } else if (f[kStatusInGap]) {
        DGN_HIP(launch_row_bounds(in.op, in.nnz, (int32_t)P, L.in_rowptr, S.status, s));
    }
    const int32_t *ops_of_out = out.op;                       // operator of every entry of out_idx
    if (out_unsorted) {
        const RowPlan plan = plan_rows(Eout, P, key_bits_for(P));
        ops_of_out = S.sorted_ops;
        if (plan.use) {
            // where tensors are numbered as they are created, this is all
            DGN_HIP(launch_bucket_rows(plan, out, true, S.status + kStatusBig + 1, S.status, S.sort_tmp, s));
            rc = enqueue_records(h, L, S.status, options, s, true, true);
            if (rc) return rc;
            rc = read_status(S.status, s, found);
            if (rc || (*found)[0] || !(*found)[kStatusPending]) return rc;
            DGN_HIP(launch_expand_rows(L.out_rowptr, (int32_t)P, (int32_t)Eout, S.sorted_ops, nullptr, nullptr, (int32_t)T, S.status, s));
            DGN_HIP(launch_clear(clr, 1, s));
        } else {
            DGN_HIP(launch_check_ids(out, S.status, s));
            DGN_HIP(launch_sort_pairs(out.op, out.tensor, S.sorted_ops, L.out_idx, Eout, key_bits_for(P), S.sort_tmp, s));
        }
        // The outputs, once in operator order and every operator's tensors ascending, get the same pass as the lists did: where
        // tensors ascend with their operators that is the order by tensor, whatever order they came in, and they need no
        // second sort.
        DGN_HIP(launch_order_rows(S.sorted_ops, L.out_idx, Eout, S.sorted_keys, S.status, s));
        const EdgeList sorted{S.sorted_ops, S.sorted_keys, Eout, (int32_t)P, (int32_t)T, nullptr, L.out_rowptr, L.prod_idx, L.prod_rowptr, L.prod1, may_run(h)};
        DGN_HIP(launch_scan_edges(nullptr, sorted, S.status, s));
        rc = enqueue_records(h, L, S.status, options, s, false);
        if (rc) return rc;
        rc = read_status(S.status, s, found);
        if (rc) return rc;
        out_gap = (*found)[kStatusOutGap];
        prod_unsorted = (*found)[kStatusProdUnsorted];
        prod_gap = (*found)[kStatusProdGap];
        if ((*found)[0] || !(out_gap || prod_unsorted || prod_gap)) return DGN_OK;
        DGN_HIP(launch_clear(order, 1, s));
    }
    // (a long gap between tensors, but their order known: the keys are the ones that were found to ascend)
    const int32_t *by_tensor = out_unsorted ? S.sorted_keys : L.out_idx;
    if (out_gap) DGN_HIP(launch_row_bounds(ops_of_out, Eout, (int32_t)P, L.out_rowptr, S.status, s));
    if (prod_unsorted || prod_gap) {
        rc = build_producers(h, L, S, ops_of_out, prod_unsorted ? nullptr : by_tensor, true, s);
        if (rc) return rc;
    }
    rc = enqueue_records(h, L, S.status, options, s, prod_unsorted || prod_gap);
    if (rc) return rc;
    return read_status(S.status, s, found);
}

// The adjacency and what follows it, from edge lists whose workspace is laid out in L and S.
int build_from_lists(dgn_graph *h, const dgn_coo_desc *d, const GraphLayout &L, const BuildScratch &S, const dgn_options *options,
                     hipStream_t s, const int32_t **found)
{
    const int64_t P = h->P, T = h->T, Ein = h->Ein, Eout = h->Eout;
    // One pass over both lists (in COO order) checks the ids, notes whether the keys ever decrease and, on the assumption
    // that they do not, already writes the finished adjacency: a graph recorded operator by operator needs nothing more,
    // and the host looks at the status once, when the records are made as well.
    int rc = copy_offsets(h, L, d->graph_op_offsets, d->graph_tensor_offsets, s);
    if (rc) return rc;
    const EdgeList in{d->in_op, d->in_tensor, Ein, (int32_t)P, (int32_t)T, L.in_idx, L.in_rowptr, nullptr, nullptr, nullptr, false};
    const EdgeList out{d->out_op, d->out_tensor, Eout, (int32_t)P, (int32_t)T, L.out_idx, L.out_rowptr, L.prod_idx, L.prod_rowptr, L.prod1, may_run(h)};
    DGN_HIP(launch_first_look(in, out, S.status, s));
    DGN_HIP(launch_scan_edges(&in, out, S.status, s));
    rc = enqueue_records(h, L, S.status, options, s, false);
    if (rc) return rc;
    rc = read_status(S.status, s, found);
    if (rc) return rc;
    int32_t f[kStatusOrder];
    for (int i = 0; i < kStatusOrder; ++i) f[i] = (*found)[i];
    if (f[0] & kErrIdRange) return DGN_OK;                    // bad ids: nothing is built from them
    if (!(f[kStatusInUnsorted] || f[kStatusInGap] || f[kStatusOutUnsorted] || f[kStatusOutGap] || f[kStatusProdUnsorted] ||
          f[kStatusProdGap]))
        return DGN_OK;
    return sort_lists(h, in, out, L, S, f, options, s, found);
}

}  // namespace

extern "C" {

int dgn_version(void) { return DGN_VERSION; }
int dgn_last_hip_error(void) { return t_last_hip; }

const char *dgn_strerror(int code)
{
    switch (code) {
        case DGN_OK: return "ok";
        case DGN_ERR_INVALID_ARG: return "invalid argument";
        case DGN_ERR_NULL_PTR: return "required pointer is NULL";
        case DGN_ERR_TOO_LARGE: return "count too large for 32-bit ids";
        case DGN_ERR_ID_OUT_OF_RANGE: return "operator, tensor or target id out of range";
        case DGN_ERR_TOO_MANY_SETS: return "number of target sets must be 1..64";
        case DGN_ERR_WORKSPACE_TOO_SMALL: return "graph storage or scratch smaller than the queried size";
        case DGN_ERR_NOT_TOPOLOGICAL: return "operator ids are not a topological order";
        case DGN_ERR_HIP: return "HIP runtime error";
        case DGN_ERR_BAD_CSR: return "malformed CSR row pointers";
        default: return "unknown error";
    }
}

int dgn_graph_build_workspace(const dgn_coo_desc *d, size_t *graph_bytes, size_t *scratch_bytes)
{
    if (!d || !graph_bytes || !scratch_bytes) return DGN_ERR_NULL_PTR;
    int rc = check_sizes(d->num_ops, d->num_tensors, d->nnz_in, d->nnz_out, d->num_graphs, d->graph_op_offsets,
                         d->graph_tensor_offsets);
    if (rc) return rc;
    *graph_bytes = graph_layout(nullptr, d->num_ops, d->num_tensors, d->nnz_in, d->nnz_out, d->num_graphs, d->graph_op_offsets, true).bytes;
    *scratch_bytes = build_scratch(nullptr, d->nnz_in, d->nnz_out).bytes;
    return DGN_OK;
}

int dgn_graph_build(const dgn_coo_desc *d, void *graph_mem, size_t graph_bytes, void *scratch, size_t scratch_bytes,
                    const dgn_options *options, dgn_stream stream, dgn_graph **out)
{
    if (!d || !out) return DGN_ERR_NULL_PTR;
    *out = nullptr;
    size_t need_g = 0, need_s = 0;
    int rc = dgn_graph_build_workspace(d, &need_g, &need_s);
    if (rc) return rc;
    rc = check_options(options);
    if (rc) return rc;
    if (!graph_mem || !scratch) return DGN_ERR_NULL_PTR;
    if ((d->nnz_in > 0 && (!d->in_op || !d->in_tensor)) || (d->nnz_out > 0 && (!d->out_op || !d->out_tensor)))
        return DGN_ERR_NULL_PTR;
    if (graph_bytes < need_g || scratch_bytes < need_s) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)graph_mem | (uintptr_t)scratch) & 7) return DGN_ERR_INVALID_ARG;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t P = d->num_ops, T = d->num_tensors, Ein = d->nnz_in, Eout = d->nnz_out;
    const GraphLayout L = graph_layout(graph_mem, P, T, Ein, Eout, d->num_graphs, d->graph_op_offsets, true);
    const BuildScratch S = build_scratch(scratch, Ein, Eout);

    dgn_graph *h = nullptr;
    rc = new_graph(&h);
    if (rc) return rc;
    h->P = P; h->T = T; h->Ein = Ein; h->Eout = Eout; h->G = d->num_graphs;
    h->v = GraphView{(int32_t)P, (int32_t)T, (int32_t)Ein, (int32_t)Eout, d->num_graphs, L.in_rowptr, L.in_idx,
                     L.out_rowptr, L.out_idx, L.prod_rowptr, L.prod_idx, nullptr, nullptr, L.orec, L.ofirst, L.prod1, -1};
    h->max_graph_ops = L.max_graph_ops;
    const int32_t *found = nullptr;
    rc = build_from_lists(h, d, L, S, options, s, &found);
    if (!rc) rc = finish_build(h, d->graph_op_offsets, d->graph_tensor_offsets, S.status, found, options, s, out);
    if (rc) delete h;
    return rc;
}

int dgn_graph_from_csr_workspace(const dgn_csr_desc *d, size_t *graph_bytes, size_t *scratch_bytes)
{
    if (!d || !graph_bytes || !scratch_bytes) return DGN_ERR_NULL_PTR;
    int rc = check_sizes(d->num_ops, d->num_tensors, d->nnz_in, d->nnz_out, d->num_graphs, d->graph_op_offsets,
                         d->graph_tensor_offsets);
    if (rc) return rc;
    *graph_bytes = graph_layout(nullptr, d->num_ops, d->num_tensors, d->nnz_in, d->nnz_out, d->num_graphs, d->graph_op_offsets, false).bytes;
    *scratch_bytes = build_scratch(nullptr, d->nnz_in, d->nnz_out).bytes;
    return DGN_OK;
}

int dgn_graph_from_csr(const dgn_csr_desc *d, void *graph_mem, size_t graph_bytes, void *scratch, size_t scratch_bytes,
                       const dgn_options *options, dgn_stream stream, dgn_graph **out)
{
    if (!d || !out) return DGN_ERR_NULL_PTR;
    *out = nullptr;
    size_t need_g = 0, need_s = 0;
    int rc = dgn_graph_from_csr_workspace(d, &need_g, &need_s);
    if (rc) return rc;
    rc = check_options(options);
    if (rc) return rc;
    if (!graph_mem || !scratch || !d->in_rowptr || !d->out_rowptr) return DGN_ERR_NULL_PTR;
    if ((d->nnz_in > 0 && !d->in_idx) || (d->nnz_out > 0 && !d->out_idx)) return DGN_ERR_NULL_PTR;
    if (graph_bytes < need_g || scratch_bytes < need_s) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)graph_mem | (uintptr_t)scratch) & 7) return DGN_ERR_INVALID_ARG;

    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t P = d->num_ops, T = d->num_tensors, Ein = d->nnz_in, Eout = d->nnz_out;
    const GraphLayout L = graph_layout(graph_mem, P, T, Ein, Eout, d->num_graphs, d->graph_op_offsets, false);
    const BuildScratch S = build_scratch(scratch, Ein, Eout);

    dgn_graph *h = nullptr;
    rc = new_graph(&h);
    if (rc) return rc;
    h->P = P; h->T = T; h->Ein = Ein; h->Eout = Eout; h->G = d->num_graphs;
    h->v = GraphView{(int32_t)P, (int32_t)T, (int32_t)Ein, (int32_t)Eout, d->num_graphs, d->in_rowptr, d->in_idx,
                     d->out_rowptr, d->out_idx, L.prod_rowptr, L.prod_idx, nullptr, nullptr, L.orec, L.ofirst, L.prod1, -1};
    h->max_graph_ops = L.max_graph_ops;
    const int32_t *found = nullptr;
    auto fill = [&]() -> int {
        FillRegion clr[1] = {{S.status, 256}};
        DGN_HIP(launch_clear(clr, 1, s));
        int e = copy_offsets(h, L, d->graph_op_offsets, d->graph_tensor_offsets, s);
        if (e) return e;
        // The borrowed arrays are checked before any kernel trusts them: what follows asks the status first, or reads a list that has no
        // valid entry then.
        DGN_HIP(launch_check_csr(h->v, S.status, s));
        // the outputs as a list in operator order: its tensors usually ascend as well, and the pass over it is all it takes
        DGN_HIP(launch_expand_rows(d->out_rowptr, (int32_t)P, (int32_t)Eout, S.sorted_ops, L.prod_idx, L.prod_rowptr, (int32_t)T, S.status, s));
        const EdgeList list{S.sorted_ops, d->out_idx, Eout, (int32_t)P, (int32_t)T, nullptr, nullptr, L.prod_idx, L.prod_rowptr, L.prod1, may_run(h)};
        DGN_HIP(launch_scan_edges(nullptr, list, S.status, s, h->G == 1));
        e = enqueue_records(h, L, S.status, options, s, false);
        if (e) return e;
        e = read_status(S.status, s, &found);
        if (e || (found[0] & (kErrCsr | kErrIdRange)) || !(found[kStatusProdUnsorted] || found[kStatusProdGap])) return e;
        e = build_producers(h, L, S, S.sorted_ops, found[kStatusProdUnsorted] ? nullptr : d->out_idx, false, s);
        if (e) return e;
        FillRegion ready[1] = {{S.status, kStatusOrder * sizeof(int32_t)}};
        DGN_HIP(launch_clear(ready, 1, s));
        e = enqueue_records(h, L, S.status, options, s, true);
        if (e) return e;
        return read_status(S.status, s, &found);
    };
    rc = fill();
    if (!rc) rc = finish_build(h, d->graph_op_offsets, d->graph_tensor_offsets, S.status, found, options, s, out);
    if (rc) delete h;
    return rc;
}

int dgn_graph_get_csr(const dgn_graph *g, const int32_t **in_rowptr, const int32_t **in_idx, const int32_t **out_rowptr,
                      const int32_t **out_idx, const int32_t **prod_rowptr, const int32_t **prod_idx)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (in_rowptr) *in_rowptr = g->v.in_rowptr;
    if (in_idx) *in_idx = g->v.in_idx;
    if (out_rowptr) *out_rowptr = g->v.out_rowptr;
    if (out_idx) *out_idx = g->v.out_idx;
    if (prod_rowptr) *prod_rowptr = g->v.prod_rowptr;
    if (prod_idx) *prod_idx = g->v.prod_idx;
    return DGN_OK;
}

int dgn_graph_get_sizes(const dgn_graph *g, int64_t *num_ops, int64_t *num_tensors, int64_t *nnz_in, int64_t *nnz_out,
                        int32_t *num_graphs)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (num_ops) *num_ops = g->P;
    if (num_tensors) *num_tensors = g->T;
    if (nnz_in) *nnz_in = g->Ein;
    if (nnz_out) *nnz_out = g->Eout;
    if (num_graphs) *num_graphs = g->G;
    return DGN_OK;
}

void dgn_graph_destroy(dgn_graph *g) { delete g; }

int dgn_prune_workspace(const dgn_graph *g, int32_t num_sets, size_t *scratch_bytes)
{
    if (!g || !scratch_bytes) return DGN_ERR_NULL_PTR;
    if (num_sets < 1 || num_sets > DGN_MAX_SETS) return DGN_ERR_TOO_MANY_SETS;
    *scratch_bytes = prune_scratch(nullptr, g->P, g->T, g->G, 0).bytes;
    return DGN_OK;
}

// Waves per graph when the ring sweep takes this call, 0 when it does not.
//   Which graphs: the sweep walks every operator, 1 024 of them in 2 us (nothing kept) to 13 us (one long chain); the level
// by level traversal costs about 4.6 us per dependent level of a thin graph and 60 to 100 us before it has done anything
// (a first prune 250 to 300 where its frontiers leave the single workgroup), but it ends where the chains do.  Up to 16 384
// operators the sweep was never the slower one for layered graphs, unrolled RNNs and sliding windows, 1 to 64 sets: 34 against
// 106 us at 800 operators, 98 against 153 at 8 400 (33 layers of 255), at worst 71 against 69 (RNN 30 wide, 15 000).  With inputs from
// all over the graph most of a group's pushes cross waves, and the line is at 4 096 (power law of 4 000: 124 against 141
// us, 4 200: 156, 137, 6 000: 235, 137).  All that with sixteen or four waves; where what is read lies so far back that
// LDS has room for one alone, it loses (35 layers of 324: 208 against 168).
//   Beyond that size it depends on what is kept, which nobody knows before.  A recorded chain of short hops (window of 64)
// of 20 000 operators: 282 against 3 300 us; an RNN as narrow, whose chains die out: 134 against 123, at 24 000 146 against 129, at
// 64 000 287 against 125, at 120 000 450 against 128.  So the line for graphs that read nothing older than 96 tensors lies where such an RNN
// loses a tenth (with a single target 87 against 74); beyond, a graph is traversed until a prune has shown that it has long
// chains: a level per 256 operators (at 4.6 us each 18 us per 1 024; the narrow RNNs take 6 to 20 levels in all).
// Several words of sets are swept in the time of one, where the traversal takes them one after the other.
//   How many waves: sixteen take a graph that has a compute unit to itself (20 000 operators in a chain of short hops:
// 0.28 ms, four waves 0.30, one 0.40); four when all graphs are resident at once that way (1 500 graphs of 20 000 operators:
// 0.95 ms, one wave 1.03, sixteen 2.13); one beyond (4 096 graphs: 1.18 ms, four waves 1.67).  Batches of 64 graphs and more
// were always swept, with hash tables and one wave per graph before, and take what fits.
// words: words of 64 sets (single graphs), a workgroup each.
static int ring_waves(const dgn_graph *g, const dgn_options *o, const dgn_stats *stats, int64_t words = 1)
{
    if (!g->ring || (o && (o->traversal != 0 || o->incremental || o->recompute_keep))) return 0;
    const bool many = g->G >= kSweepMinGraphs;               // (such batches were always swept graph by graph)
    if (!many && stats && stats->level_trace && stats->level_trace_cap > 0) return 0;     // asks for levels: there are none here
    const bool thin = g->ring_dist <= kRingThinDist;
    int64_t most = thin ? kRingThinOps : g->reads_about ? kRingAboutOps : kRingShortOps;
    most = words > kRingMaxOps / most ? kRingMaxOps : most * words;
    if (!thin && most > kRingShortOps) most = kRingShortOps;
    if (thin && g->long_chains.load(std::memory_order_relaxed)) most = kRingMaxOps;
    if (many) most = kRingMaxGraphOps;
    if (g->max_graph_ops > most) return 0;
    auto fits = [&](int w) {
        return ((size_t)ring_words(w, g->ring_dist, g->ring_span64) + (size_t)g->ring_low + kRingExtraWords) * sizeof(u64) +
                   kRingSeedWords * sizeof(uint32_t) <= kRingMaxLds;
    };
    const int64_t groups = g->G > 1 ? g->G : words;
    if (groups <= g->num_cus && g->max_graph_ops > 4 * kWave) {
        if (fits(16)) return 16;
        if (!many) return fits(4) ? 4 : 0;
    }
    if (groups <= 8 * g->num_cus && fits(4)) return 4;
    return fits(1) ? 1 : 0;
}

// Segments per graph of a ring sweep (laid out in a, in `room`), 1: none.
//   A graph that is read at most 64 tensors back may be swept in pieces at the same time: what a piece does not know is M of
// the 64 tensors below its upper end, and it is linear in those, so a second sweep whose sets are those tensors says what they
// bring (see ring_sweep.hip).  A chain of 0.9 us per 64 operators becomes two sweeps of a few words each, side by side, 10 to 17 us to
// put them together, and twice the work.  Whole prunes, in one piece / in segments: one graph of 500
// operators 36.5 / 34.5 us, 2 000 50 / 34.5, 20 000 284 / 50; 150 sets on 20 000 292 / 50; 20 graphs of up to 5 100 operators 98 / 54,
// 96 of them 97 / 54, 250 graphs of 20 000 309 / 230.  The work (50 ps per operator and two sweeps of it) is what it loses by: 500 graphs of 3 000
// 86 / 95, 1 000 of 6 000 217 / 302.
//   Two words of 64 operators per segment up to 1 024 operators, four beyond (2 000: 34.5 us, eight 37; 800: two 35.4, four 37.1); not
// more than 64 segments (20 000: 52.4 us with 79, 50 with 40), nor than 24 waves of sweeps per compute unit (250 graphs of 20 000: 8 words per
// segment 271 us, 16 248, 32 230); and what has room.
//   Every segment looks at all targets of its graph.  With up to two workgroups per compute unit (one, if the targets go by way of
// M) eight waves each do (2 000 operators: 8 192 targets 66 us in one piece / 49, one wave 91; 64 000 112 / 96, 411; 40 graphs of 800 with
// 4 096 each 73 / 69, 78), else the one that sweeps: more of them are in each other's way (250 graphs of 5 000, 256 targets each: 148 /
// 91, eight 118).  What is gained then was fitted to 250 batches of 8 to 600 graphs, with 2 us in its favour: the chain without that
// of a segment, less the operators and the targets (250 graphs of 1 000, which have room for two segments each, 1 024 targets: 59 /
// 66).  More than kRingSeedWords targets go by way of M, which is slow in one piece as well (250 graphs of 1 000, 4 096 each: 161 / 105; 96
// of 3 000: 16 384 188 / 188, 25 600 219 / 293).
static int ring_segments(const dgn_graph *g, int64_t words, Room room, RingArgs &a)
{
    if (g->ring_reach > kWave) return 1;
    const int64_t n_words = (g->max_graph_ops + kWave - 1) / kWave, all_words = (g->P / kWave + 1) * (words + 1);
    const double swept = (double)g->P * (double)(words + 1);
    if ((double)n_words * kRingWordUs < kRingSegmentsUs + swept * kRingSegmentOpUs) return 1;
    int shift = n_words <= kRingFewWords ? 1 : 2;
    while ((n_words >> shift) > kRingManySegs || (all_words >> shift) > kRingSegmentsPerCu * g->num_cus) ++shift;
    for (;; ++shift) {
        a.seg_shift = shift;
        a.seg_words = 1 << shift;
        const int64_t segs = (n_words + a.seg_words - 1) >> shift;
        if (segs < 2 || a.seg_words > kRingMaxSegWords) return 1;
        a.segs = (int32_t)segs;
        if (ring_segment_scratch(a, nullptr) <= room.bytes) break;
    }
    const int64_t targets = a.num_targets / (g->G * words);  // (of an average graph or word)
    const bool from_m = targets > kRingSeedWords;
    a.few_segs = (int64_t)g->G * a.segs * (words + 1) <= (int64_t)(from_m ? 1 : kRingFewSegmentsPerCu) * g->num_cus;
    const double targets_us = from_m ? (double)targets * kRingFromMTargetUs - kRingFromMUs : (double)targets * kRingManyTargetUs;
    if (!a.few_segs && (double)n_words * kRingManyWordUs + kRingManyUs <
                           (double)a.seg_words * kRingManySegWordUs + swept * kRingManyOpUs + targets_us)
        return 1;
    (void)ring_segment_scratch(a, room.at);
    return a.segs;
}

// dgn_prune of graphs that the ring sweep takes: one to three launches, nothing to clear beforehand.
// words > 1: as many words of 64 sets of a single graph at once, num_sets in all.  S.flagbuf == NULL: no flag bytes but
// the caller's are kept.
static int ring_prune(const dgn_graph *g, int waves, int64_t words, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
                      const int32_t *tgt_idx, u64 *M, u64 *K, uint8_t *op_flag, int32_t *kept_ops, u64 *kept_masks,
                      int64_t *kept_count, int64_t *per_query_count, const PruneScratch &S, const dgn_options *options,
                      dgn_stats *stats, hipStream_t s, u64 *also_M, u64 *also_K)
{
    void *pin = nullptr;
    int rc = pinned_buffer(&pin);
    if (rc) return rc;
    // 0 start, 1 cleared, 2 swept, 3 counted (batches), 4 listed; profile = 2: those around the sweep alone
    hipEvent_t *ev = nullptr;
    const bool all = options && options->profile == 1;
    int launches = 0;
    if (options && options->profile && stats) {
        rc = profile_events(&ev);
        if (rc) return rc;
        if (all) DGN_HIP(hipEventRecord(ev[0], s));
    }
    if (also_M || also_K) {
        FillRegion more[2] = {{also_M, (size_t)g->T * 8}, {also_K, (size_t)g->P * 8}};
        DGN_HIP(launch_clear(more, 2, s));
        ++launches;
    }
    uint8_t *flags = ring_flags(S, op_flag, g->P);
    RingArgs a{};
    a.g = g->v;
    a.num_sets = num_sets;
    a.words = (int32_t)words;
    a.num_targets = num_targets;
    a.tgt_rowptr = tgt_rowptr;
    a.tgt_idx = tgt_idx;
    a.M = M;
    a.K = K;
    a.flags = flags;
    a.flags2 = flags == op_flag ? nullptr : op_flag;
    a.kept_ops = kept_ops;
    a.kept_masks = kept_masks;
    a.kept_count = kept_count;
    a.pq = per_query_count;
    a.bits = S.ring_bits;
    a.cum = S.ring_cum;
    a.graphs = S.ring_graphs;
    a.host_status = static_cast<int32_t *>(pin);
    a.hdr = S.hdr;
    a.want = RecycleHeader{kRingMagic, g->serial, M, K, kept_ops, kept_count, flags, nullptr, nullptr, {0, 0, 0}};
    // (many graphs: nearly every word of a batch is written anyway, and the flag has no effect)
    a.recycle = options && options->recycle && g->G < kSweepMinGraphs;
    a.low_words = g->ring_low;
    // targets of a graph that fit in LDS; a graph with more of them sends its targets through M
    const int64_t avg = num_targets / g->G;
    a.seed_words = (int32_t)(g->G == 1 /* a word may own any part of them */ ? (avg < kRingSeedWords ? avg : kRingSeedWords)
                                       : (avg + avg / 2 + 64 < kRingSeedWords ? avg + avg / 2 + 64 : kRingSeedWords));
    a.reach = g->ring_reach;
    a.count_steps = stats && g->G < kSweepMinGraphs;
    a.segs = ring_segments(g, words, segments_room(S, words), a);
    if (a.segs > 1 && a.seed_words < kWave) a.seed_words = kWave;
    int32_t *status = static_cast<int32_t *>(pin);
    status[0] = status[1] = status[2] = 0;
    if (ev) DGN_HIP(hipEventRecord(ev[1], s));
    int sweep_launches = 0;
    DGN_HIP(launch_ring_sweep(a, waves, g->ring_dist, g->ring_span64, g->max_graph_ops, &sweep_launches, s, ev ? ev + 2 : nullptr, all));
    launches += sweep_launches;
    DGN_HIP(hipStreamSynchronize(s));
    if (stats) {
        int32_t *user_trace = stats->level_trace;
        const int64_t user_cap = stats->level_trace_cap;
        memset(stats, 0, sizeof(*stats));
        stats->level_trace = user_trace;
        stats->level_trace_cap = user_cap;
        stats->launches = launches;
        stats->levels = g->G < kSweepMinGraphs ? status[1] : 0;
        stats->tensor_visits = g->P * words;
        stats->recycled = status[2];
        if (ev) {
            DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TRAVERSE], ev[1], ev[2]));
            if (all) {
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_CLEAR], ev[0], ev[1]));
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_SCAN], ev[2], ev[3]));
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_SCATTER], ev[3], ev[4]));
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TOTAL], ev[0], ev[4]));
            }
        }
    }
    return error_bits_to_code(status[0]);
}

// The largest graph that is swept by layers, for so many sets and targets (see kBandSoonShare).  The last word of several goes by its
// own sets as well (65 sets, 1 000 x 800 1 284 us with that one set swept, 1 065 with it left to the levels, 500 x 700 667 / 579, 300 x 667
// 430 / 402, but 1 000 x 210 577 / 666, 1 000 x 300 640 / 715, 800 x 500 653 / 656).
static int64_t band_most_ops(const dgn_graph *g, int64_t sets, int64_t num_targets, bool last_word)
{
    const bool deep = g->reach == Reach::nearer;
    if (num_targets > kBandMaxTargets) {
        const bool many = sets >= kBandFromMManySets || (sets > kBandFewSets && deep);
        return many ? kBandFromMMaxOps : kBandFromMOps + sets * kBandFromMSetOps;
    }
    return sets > kBandFewSets ? kBandMaxOps : !deep ? kBandFewSetsOps : last_word ? kBandLastWordDeepOps : kBandFewSetsDeepOps;
}

// dgn_prune of a graph that looks like layers (see band_sweep.hip).  *taken: whether it was one; if not, nothing but a clear has
// happened.  *launches: kernels enqueued.
static int band_prune(const dgn_graph *g, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr, const int32_t *tgt_idx,
                      u64 *M, u64 *K, uint8_t *op_flag, int32_t *kept_ops, u64 *kept_masks, int64_t *kept_count,
                      int64_t *per_query_count, const PruneScratch &S, const dgn_options *options, dgn_stats *stats, hipStream_t s,
                      u64 *also_M, u64 *also_K, bool *taken, int64_t *launches)
{
    *taken = false;
    *launches = 0;
    BandArgs a{};
    a.g = g->v;
    if (reinterpret_cast<const char *>(S.q0) + band_scratch(a, nullptr) > reinterpret_cast<const char *>(S.flagbuf)) return DGN_OK;
    (void)band_scratch(a, S.q0);
    void *pin = nullptr;
    int rc = pinned_buffer(&pin);
    if (rc) return rc;
    // 0 start, 1 cleared, 2 seeded, 3 swept, 4 counted, 5 scanned, 6 listed; profile = 2: those around the sweep alone
    hipEvent_t *ev = nullptr;
    const bool all = options && options->profile == 1;
    if (options && options->profile && stats) {
        rc = profile_events(&ev);
        if (rc) return rc;
        if (all) DGN_HIP(hipEventRecord(ev[0], s));
    }
    const size_t pq_bytes = per_query_count ? sizeof(int64_t) * 64 : 0;
    a.num_sets = num_sets;
    a.num_targets = num_targets;
    a.tgt_rowptr = tgt_rowptr;
    a.tgt_idx = tgt_idx;
    a.M = M;
    a.state = S.state;
    a.host_status = static_cast<int32_t *>(pin);
    a.hdr = S.hdr;
    a.want = RecycleHeader{kBandMagic, g->serial, M, K, kept_ops, kept_count, op_flag, also_M, also_K, {0, 0, 0}};
    a.recycle = options && options->recycle;
    for (int i = 0; i < 8; ++i) a.host_status[i] = 0;
    const FillRegion clear[kBandRegions] = {{M, (size_t)g->T * 8}, {S.state, 256 + sizeof(TravCounters)},
                                            {per_query_count, pq_bytes}, {S.pq_part, per_query_count ? S.pq_part_bytes : 0},
                                            {also_M, (size_t)g->T * 8}, {also_K, (size_t)g->P * 8}};
    for (int i = 0; i < kBandRegions; ++i) a.clear[i] = clear[i];
    const bool from_m = num_targets > kBandMaxTargets;
    // (the backward prune goes on with the flag bytes where the traversal would have kept them)
    uint8_t *flags = also_M ? ring_flags(S, op_flag, g->P) : op_flag;
    if (flags != op_flag) {
        FillRegion more[1] = {{flags, S.db_bytes}};
        DGN_HIP(launch_clear(more, 1, s));
        ++*launches;
    }
    DGN_HIP(launch_band_plan(a, g->num_cus, s));
    if (ev && all) DGN_HIP(hipEventRecord(ev[1], s));
    if (from_m) DGN_HIP(launch_seed(g->v, num_sets, num_targets, tgt_rowptr, tgt_idx, M, S.state, S.ctr, nullptr, S.qg, 0, ColourLog{}, s));
    if (ev) DGN_HIP(hipEventRecord(ev[2], s));
    DGN_HIP(launch_band_sweep(a, from_m, s));
    if (ev) DGN_HIP(hipEventRecord(ev[3], s));
    CompactArgs ca{};
    ca.g = g->v;
    ca.M = M;
    ca.K = K;
    ca.op_flag = op_flag ? op_flag : flags;
    ca.from_tensor_mask = true;                             // (of M and K the sweep writes M only)
    ca.kept_ops = kept_ops;
    ca.kept_masks = kept_masks;
    ca.kept_count = kept_count;
    ca.per_query_count = per_query_count;
    ca.opbits = S.opbits;
    ca.block_counts = S.block_counts;
    ca.pq_part = S.pq_part;
    ca.pq_replicas = S.pq_replicas;
    ca.hdr = a.recycle ? S.hdr : nullptr;
    ca.want = a.want;
    ca.error = &S.state->error;
    DGN_HIP(launch_keep_compact(ca, s, ev && all ? ev + 4 : nullptr));
    if (op_flag && flags != op_flag) DGN_HIP(hipMemcpyAsync(flags, op_flag, (size_t)g->P, hipMemcpyDeviceToDevice, s));
    *launches += from_m ? 6 : 5;                            // plan, seeds, sweep, count, scan, list
    DGN_HIP(hipStreamSynchronize(s));
    const int32_t *status = a.host_status;
    if (status[kBandTaken] == 0) {
        g->no_layers.store(1, std::memory_order_relaxed);
        return DGN_OK;
    }
    *taken = true;
    if (stats) {
        int32_t *user_trace = stats->level_trace;
        const int64_t user_cap = stats->level_trace_cap;
        memset(stats, 0, sizeof(*stats));
        stats->level_trace = user_trace;
        stats->level_trace_cap = user_cap;
        stats->launches = *launches;
        stats->levels = status[kBandTaken] - 1;
        stats->tensor_visits = g->P;
        stats->recycled = status[kBandFound];
        if (ev && all) {
            for (int i = 0; i < 6; ++i) DGN_HIP(hipEventElapsedTime(&stats->phase_ms[i], ev[i], ev[i + 1]));
            DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TOTAL], ev[0], ev[6]));
        } else if (ev) {
            DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TRAVERSE], ev[2], ev[3]));
        }
    }
    return error_bits_to_code(status[kBandErrors] | status[kBandErrors + 1] | status[kBandErrors + 2] | status[kBandErrors + 3]);
}

// What dgn_prune asks of its arguments; lays out its scratch.
static int check_prune(const dgn_graph *g, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
                       const int32_t *tgt_idx, const uint64_t *tensor_mask, const uint64_t *op_mask, const int32_t *kept_ops,
                       const uint64_t *kept_masks, const int64_t *kept_count, const int64_t *per_query_count, void *scratch,
                       size_t scratch_bytes, const dgn_options *options, PruneScratch *S, bool whole_queues = false)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (num_sets < 1 || num_sets > DGN_MAX_SETS) return DGN_ERR_TOO_MANY_SETS;
    if (num_targets < 0) return DGN_ERR_INVALID_ARG;
    if (num_targets > kMaxCount) return DGN_ERR_TOO_LARGE;
    const int rc = check_options(options);
    if (rc) return rc;
    if (!tgt_rowptr || (num_targets > 0 && !tgt_idx) || !kept_count || !scratch) return DGN_ERR_NULL_PTR;
    if ((g->T > 0 && !tensor_mask) || (g->P > 0 && (!op_mask || !kept_ops))) return DGN_ERR_NULL_PTR;
    *S = prune_scratch(scratch, g->P, g->T, g->G, options ? options->max_queue_entries : 0, whole_queues);
    if (scratch_bytes < S->bytes) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)scratch | (uintptr_t)tensor_mask | (uintptr_t)op_mask | (uintptr_t)kept_masks |
         (uintptr_t)kept_count | (uintptr_t)per_query_count) & 7)
        return DGN_ERR_INVALID_ARG;
    return DGN_OK;
}

// Launches enqueued before anything is known of a graph's levels.  One that finds nothing costs 2.4 us, a group of twelve wide
// ones and the single-workgroup kernel 30; a batch that falls short a wait, a compaction for nothing and another group, 90 to 120.
// Power-law graphs of up to half a million operators take 8 to 14 levels (300 000 operators, 64 sets, first prune: four groups 327
// us, two 271, one 234; 1 M takes 13 to 16: 360, 300, 379), graphs of 218 to 750 layers 9 to 13 wide ones (500 x 400: 474, 409, 380), and
// small graphs of any kind fit more often than not (120 x 200: 309, 250, 220; 1 000 x 40, the deepest: 487, 428, 473).
// Others, 120 x 600 (359, 305, 404), 900 x 300 (590, 522, 576), an RNN of 400 000 (824, 761, 813), take two.
static int first_groups(const dgn_graph *g)
{
    const bool few = g->P <= kOneGroupOps || g->reach == Reach::near || (g->reach == Reach::unknown && g->P <= kOneGroupFlatOps);
    return few ? 1 : 2;
}

// dgn_prune.  also_M [T] / also_K [P] (or NULL): two more arrays that the call zeroes with M and K -- all of them,
// or, with recycled buffers, the words that the previous call's log and kept list name (the caller vouches that
// they hold non-zero words nowhere else).  Such a caller goes on to use the queues' room for lists of its own.
// sets, targets: what the schedule goes by: num_sets and num_targets, or, for a word of several, those of an average word (the
// same for all, so that they take the same launches: 45 layers of 340, 120 sets of 4 or 5, 320 us, each by its own 420).
static int prune_impl(const dgn_graph *g, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
                      const int32_t *tgt_idx, uint64_t *tensor_mask, uint64_t *op_mask, uint8_t *op_flag, int32_t *kept_ops,
                      uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count, void *scratch,
                      size_t scratch_bytes, const dgn_options *options, dgn_stats *stats, dgn_stream stream,
                      uint64_t *also_M, uint64_t *also_K, int64_t sets, int64_t targets)
{
    PruneScratch S{};
    int rc = check_prune(g, num_sets, num_targets, tgt_rowptr, tgt_idx, tensor_mask, op_mask, kept_ops, kept_masks, kept_count,
                         per_query_count, scratch, scratch_bytes, options, &S, also_M != nullptr);
    if (rc) return rc;

    hipStream_t s = static_cast<hipStream_t>(stream);
    u64 *M = reinterpret_cast<u64 *>(tensor_mask);
    u64 *K = reinterpret_cast<u64 *>(op_mask);
    const int ring = ring_waves(g, options, stats);
    if (ring)
        return ring_prune(g, ring, 1, num_sets, num_targets, tgt_rowptr, tgt_idx, M, K, op_flag, kept_ops,
                          reinterpret_cast<u64 *>(kept_masks), kept_count, per_query_count, S, options, stats, s,
                          reinterpret_cast<u64 *>(also_M), reinterpret_cast<u64 *>(also_K));
    const bool plain = !(options && (options->traversal != 0 || options->incremental || options->recompute_keep)) &&
                       !(stats && stats->level_trace && stats->level_trace_cap > 0);
    int64_t launches = 0, level_launches = 0;
    if (g->layers && plain && g->P <= band_most_ops(g, num_sets, num_targets, num_sets < sets) && !g->no_layers.load(std::memory_order_relaxed)) {
        bool taken = false;
        rc = band_prune(g, num_sets, num_targets, tgt_rowptr, tgt_idx, M, K, op_flag, kept_ops, reinterpret_cast<u64 *>(kept_masks),
                        kept_count, per_query_count, S, options, stats, s, reinterpret_cast<u64 *>(also_M),
                        reinterpret_cast<u64 *>(also_K), &taken, &launches);
        if (rc || taken) return rc;
    }
    const size_t pq_bytes = per_query_count ? sizeof(int64_t) * 64 * (size_t)(g->G > 1 ? g->G : 1) : 0;
    // 0 start, 1 cleared, 2 seeded, 3 traversed, 4 counted, 5 scanned, 6 scattered.  An event between two
    // kernels costs a few microseconds of idle stream, so profile = 2 records only the two around the traversal.
    hipEvent_t *ev = nullptr;
    hipEvent_t *ev_trav = nullptr;
    if (options && options->profile && stats) {
        rc = profile_events(&ev_trav);
        if (rc) return rc;
        if (options->profile == 1) {
            ev = ev_trav;
            DGN_HIP(hipEventRecord(ev[0], s));
        }
    }

    // nothing marked yet: clear outputs, deferral markers and traversal state (an incremental call keeps
    // M and K: they hold a fixed point that the new target bits only add to).  With `recycle` the scratch
    // buffer may say that M, K and the kept list are still those of the previous prune of this graph: then
    // only what that prune set is zeroed, and this prune keeps a log of what it colours for the next one.
    const bool incremental = options && options->incremental;
    const bool sweep = !(options && options->traversal != 0) && is_swept(g->G, g->max_graph_ops) && g->topological;
    const bool recycle = options && options->recycle && !incremental && !sweep && g->P > 0;
    // The traversal sets a byte for every operator whose K leaves zero, which lets the count pass read P bytes
    // and the K of the kept operators instead of all of K.  The bytes are the caller's op_flag when that can be
    // cleared in whole 8-byte words, else a scratch array.  (Not for the per-graph sweep, which writes K
    // without atomics and finds nothing out about "first"; not for incremental calls, whose K comes from outside.)
    const bool use_flags = !sweep && !incremental && !(options && options->recompute_keep);
    uint8_t *flags = (op_flag && ((uintptr_t)op_flag & 7) == 0 && g->P % 8 == 0) ? op_flag : S.flagbuf;
    const size_t flag_bytes = flags == op_flag ? (size_t)g->P : S.db_bytes;
    const ColourLog log{recycle ? S.log.entries : nullptr, S.log.cnt, S.log.seg_cap};
    const RecycleHeader want{kRecycleMagic, g->serial, M, K, kept_ops, kept_count, flags, also_M, also_K, {0, 0, 0}};
    if (recycle) {
        // (the flag bytes are cleared whether or not this call's count pass reads them: the header this call leaves
        // names them, and the call that finds it zeroes them at this call's kept operators only)
        FillRegion big[6] = {{M, (size_t)g->T * 8}, {K, (size_t)g->P * 8}, {S.DB, S.db_bytes},
                             {flags, flag_bytes}, {also_M, (size_t)g->T * 8}, {also_K, (size_t)g->P * 8}};
        DGN_HIP(launch_clear_or_reset(big, 6, S.hdr, want, reinterpret_cast<u64 *>(S.state + 1), S.log, kept_ops, kept_count, M, K,
                                      S.DB, flags, s));
        // (the word behind the state header says which way the kernel above went: it comes back with the header)
        FillRegion small[6] = {{S.state, sizeof(TravState)}, {S.ctr, sizeof(TravCounters)}, {S.hdr, sizeof(RecycleHeader)},
                               {S.log.cnt, sizeof(SegCounter) * kMaxSeg}, {per_query_count, pq_bytes},
                               {S.pq_part, per_query_count ? S.pq_part_bytes : 0}};
        DGN_HIP(launch_clear(small, 6, s));
        ++launches;
    } else {
        // (the per-graph sweep stores K of every operator and uses no markers: it needs M cleared, nothing else)
        FillRegion clr[8] = {{M, incremental ? 0 : (size_t)g->T * 8}, {K, incremental || sweep ? 0 : (size_t)g->P * 8},
                             {S.DB, sweep ? 0 : S.db_bytes}, {S.state, 256 + sizeof(TravCounters)}, {S.hdr, 256},
                             {per_query_count, pq_bytes}, {S.pq_part, per_query_count ? S.pq_part_bytes : 0},
                             {flags, use_flags ? flag_bytes : 0}};
        DGN_HIP(launch_clear(clr, 8, s));
        if (also_M || also_K) {
            FillRegion more[2] = {{also_M, (size_t)g->T * 8}, {also_K, (size_t)g->P * 8}};
            DGN_HIP(launch_clear(more, 2, s));
            ++launches;
        }
    }
    if (ev) DGN_HIP(hipEventRecord(ev[1], s));
    // Deferral schedule: threshold on the producer id, starting at decay*P and decaying geometrically down to a floor.  Bits
    // that keep coming from above are worth waiting for; below the floor, one launch takes the rest, in which
    // operators are processed again and again, but a launch costs 14 us at least.
    //   P >> 10 loses nowhere: higher floors are faster for some targets of a power-law graph and slower for others
    // (400 000 operators, 2 sqrt(P): 64 sets of one target 196 -> 233 us, of 8 223 -> 207).  From 4 M operators on 2 sqrt(P) is the
    // lower one, and never slower (20 M, one set of 8: 320 -> 252; 50 M, 64 sets: 662 -> 643; backward prune 1 001 -> 921).
    //   Where operators read what was written shortly before, bits come soon one after the other, and waiting for thresholds
    // far below only makes the levels thin: P >> 3 for 200 000 operators in 500 layers, 64 sets 405 -> 300 us, for
    // 702 000 in 900 layers 1 123 -> 740, for 18 000 in 300 layers 262 -> 190.  The line lies at some 218 layers, each reading
    // mostly the one before: with 100 layers and a handful of targets what is left below P >> 3 is too little to
    // spread over the chip (300 wide, 8 targets: 152 us, P >> 3 310), with 200 it still is for some (800 wide: 332, 412).
    //   With some 700 to 800 layers and more it depends on how wide the levels are.  One set, 892 layers: 298 wide 375 us,
    // P >> 3 410; 500 wide 415, 425; 1 000 layers of 600: 648, 477.  Four sets: 200 wide 426, 440; 300 wide 525, 471.  Eight:
    // 100 wide 400, 406; 156 wide 425, 416.  So the line lies at 450 000 operators over the root of the sets; beyond eight
    // sets P >> 3 was never the slower one (17 sets, 100 wide 450, 424; 64 sets, 50 wide 403, 386; RNN of 20 000, 64 sets 128, 110).
    //   From some 30 layers on, it pays as well once there are many targets: at 224 and more P >> 3 was the faster one for each of six
    // shapes (120 layers of 600, 288 targets 307 -> 249), around 150 not for all (264, 286).
    //   In a graph thousands of levels deep a few hundred targets all over it are as many separate searches, and the
    // thresholds let them run side by side: an RNN of 1 M operators, 70 targets 348 us, the short way 471, 10 M and
    // 33 targets 236, 333; with many targets the short way is the better one (544 of them: 80 000 operators 183 -> 137,
    // 200 000 190 -> 134, 450 000 907 -> 753, 800 000 286 -> 225; larger ones not tried).
    const int defer_percent = options && options->defer_percent ? options->defer_percent : kDefaultDeferPercent;
    const int start_shift = options && options->defer_start_shift ? options->defer_start_shift : kDefaultStartShift;
    Schedule sch{1.0f, 0, 0, kSmallLevel};
    if (defer_percent < 100) {
        sch.decay = (float)defer_percent / 100.0f;
        sch.theta0 = (int32_t)(g->P >> start_shift);
        const bool soon = g->reach == Reach::near ||
                          (g->reach == Reach::nearer &&
                           (sets > kFewSets || (double)g->P * (double)g->P * (double)sets > kFewSetsOps * kFewSetsOps)) ||
                          (g->reach == Reach::layers && targets >= kLayeredTargets) ||
                          (g->reach == Reach::deep && targets >= kDeepTargets && g->P <= kDeepOps);
        sch.theta_floor = (int32_t)(g->P >> (soon ? kNearFloorShift : kDefaultFloorShift));
        if (g->reach < Reach::deep && !soon) {
            const double root = kDefaultFloorPerRoot * sqrt((double)g->P);
            if (root < sch.theta_floor) sch.theta_floor = (int32_t)root;
        }
        if (options && options->defer_floor_shift) sch.theta_floor = (int32_t)(g->P >> options->defer_floor_shift);
        if (sch.theta_floor < 64) sch.theta_floor = 64;
        if (sch.theta0 < sch.theta_floor) sch.theta0 = 0;
    }
    DGN_HIP(launch_seed(g->v, num_sets, num_targets, tgt_rowptr, tgt_idx, M, S.state, S.ctr, sweep ? nullptr : S.q0, S.qg,
                        sch.theta0, log, s));
    if (ev_trav) DGN_HIP(hipEventRecord(ev_trav[2], s));
    launches += 2;

    CompactArgs ca{};
    ca.g = g->v;
    ca.M = M;
    ca.K = K;
    ca.op_flag = op_flag;
    ca.kept_ops = kept_ops;
    ca.kept_masks = reinterpret_cast<u64 *>(kept_masks);
    ca.kept_count = kept_count;
    ca.per_query_count = per_query_count;
    ca.opbits = S.opbits;
    ca.block_counts = S.block_counts;
    ca.pq_part = S.pq_part;
    ca.pq_replicas = S.pq_replicas;
    ca.from_tensor_mask = options && options->recompute_keep;
    ca.flag_in = use_flags ? flags : nullptr;
    ca.hdr = recycle ? S.hdr : nullptr;
    ca.want = want;
    ca.error = &S.state->error;

    void *pin = nullptr;
    rc = pinned_buffer(&pin);
    if (rc) return rc;
    const TravState *hst = static_cast<const TravState *>(pin);

    // Packed batch of many small graphs in topological order: one wave sweeps each graph once (see
    // k_sweep_graphs); no frontier, no level loop, per-set counts come out of the sweep itself.
    if (sweep) {
        DGN_HIP(launch_sweep_graphs(g->v, M, K, ca.from_tensor_mask ? nullptr : per_query_count, g->multi_producer, s));
        ++launches;
        if (ev_trav) DGN_HIP(hipEventRecord(ev_trav[3], s));
        if (!ca.from_tensor_mask) ca.per_query_count = nullptr;   // already written by the sweep
        DGN_HIP(launch_keep_compact(ca, s, ev ? ev + 4 : nullptr));
        launches += 3 + (g->G > 1);
        DGN_HIP(hipMemcpyAsync(pin, S.state, sizeof(TravState), hipMemcpyDeviceToHost, s));
        DGN_HIP(hipStreamSynchronize(s));
        if (stats) {
            int32_t *user_trace = stats->level_trace;
            const int64_t user_cap = stats->level_trace_cap;
            memset(stats, 0, sizeof(*stats));
            stats->level_trace = user_trace;
            stats->level_trace_cap = user_cap;
            stats->launches = launches;
            stats->tensor_visits = g->P;
            if (ev) {
                for (int i = 0; i < 6; ++i) DGN_HIP(hipEventElapsedTime(&stats->phase_ms[i], ev[i], ev[i + 1]));
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TOTAL], ev[0], ev[6]));
            } else if (ev_trav) {
                DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TRAVERSE], ev_trav[2], ev_trav[3]));
            }
        }
        return error_bits_to_code(hst->error & ~kErrOverflow);
    }

    // Level loop.  The number of levels depends on the data, so the host enqueues kernels ahead and
    // reads the 64-byte state back at a few points:
    //   1. one single-workgroup launch walks all leading small levels (deep, thin graphs finish here);
    //   2. otherwise batches of wide levels with a single-workgroup launch after every few of them; the
    //      removal-rule/compaction passes are enqueued right behind the first batch and redone only if
    //      the traversal turns out unfinished.
    int grid = g->num_cus * kLevelBlocksPerCU;
    const int64_t max_useful = (g->T + 255) / 256;
    if (grid > max_useful) grid = (int)(max_useful > 0 ? max_useful : 1);
    const bool generic_only = options && options->traversal == 1;
    const int hk = (options && options->incremental) ? 1 : 0;      // which set of layout hints
    const int small_frontier = g->reach >= Reach::near ? kNarrowCapNear : kNarrowCap;
    const int narrow_cap = generic_only ? 0 : small_frontier;
    int launch_no = 0;
    int32_t *user_trace = stats ? stats->level_trace : nullptr;
    const int64_t user_trace_cap = stats ? stats->level_trace_cap : 0;
    Quad *trace = (user_trace && user_trace_cap > 0) ? S.trace : nullptr;
    // the stand-alone removal-rule pass rewrites K, which the traversal still needs while unfinished
    const bool speculate = !ca.from_tensor_mask;
    bool done = false, compacted = false;
    // The record of a single-workgroup launch is a complete state (it leaves no tallies to fold in), so every
    // batch ends with one, and that record is what is read back.
    bool last_was_narrow = false;
    auto narrow = [&](int cap) -> int {
        DGN_HIP(launch_narrow(g->v, S.state, S.ctr, launch_no, S.q0, S.q1, S.qg, S.DB, flags, M, K, cap, sch, log, trace, s));
        ++launch_no; ++launches;
        last_was_narrow = true;
        return DGN_OK;
    };
    auto read_state = [&]() -> int {
        if (!last_was_narrow) {
            const int e = narrow(narrow_cap);
            if (e) return e;
        }
        DGN_HIP(hipMemcpyAsync(pin, S.state, 2 * sizeof(TravState), hipMemcpyDeviceToHost, s));
        DGN_HIP(hipStreamSynchronize(s));
        const LevelSlot &sl = hst->slot[(launch_no - 1) & 1];
        done = sl.n == 0 && !(sl.deferred_seen && sl.theta_hi > 0);
        return DGN_OK;
    };
    // A graph that needed wide levels last time starts with them at once: the wide kernel's second hop takes
    // the first two levels in one launch, where the single-workgroup kernel would stop after the first.
    const bool starts_wide = generic_only || g->wide_hint[hk].load(std::memory_order_relaxed) != 0;
    if (!starts_wide) {
        rc = narrow(kNarrowCap);
        if (rc) return rc;
        rc = read_state();
        if (rc) return rc;
    }
    auto group = [&](int levels) -> int {            // `levels` wide launches, then the single-workgroup kernel
        for (int i = 0; i < levels; ++i) {
            // (a traversal that starts with a wide launch: that launch takes the seeds' level however small it is)
            const int cap = launch_no == 0 ? 0 : narrow_cap;
            DGN_HIP(launch_level(g->v, S.state, S.ctr, launch_no, S.q0, S.q1, S.qg, S.DB, flags, M, K, grid, cap, sch, log, trace, s));
            ++launch_no; ++launches; ++level_launches;
        }
        last_was_narrow = false;
        return narrow(narrow_cap);
    };
    bool first = true;
    int batch = 0;
    int used_runs = 0, used_len[kMaxRuns] = {};       // the layout enqueued from the hints, if any
    while (!done) {
        const int hint_runs = generic_only ? 0 : g->hint_runs[hk].load(std::memory_order_relaxed);
        if (first && hint_runs > 0) {
            // the layout the previous prune of this graph turned out to need, plus a short tail
            int room = kMaxBatch;
            for (int r = 0; r < hint_runs && r < kMaxRuns && room > 0; ++r) {
                int len = g->hint_run_len[hk][r].load(std::memory_order_relaxed);
                len = len < 1 ? 1 : len > room ? room : len;
                rc = group(len);
                if (rc) return rc;
                room -= len + 1;
                used_len[used_runs++] = len;
            }
            if (g->exact_streak[hk].load(std::memory_order_relaxed) < kExactStreak) {
                rc = group(kTailLevels);
                if (rc) return rc;
            }
        } else {
            // unknown graph, or the layout fell short: groups of wide levels with the single-workgroup kernel
            // after each; a batch right after a hinted one is small (the hint was nearly right)
            const bool learns = first && starts_wide && !generic_only;     // (one workgroup did all of the call before)
            const int doubled = batch < 4 ? 1 << (batch > 0 ? batch - 1 : 0) : kWideGroups;
            const int groups = learns ? 1 : first ? first_groups(g) : doubled;
            for (int i = 0; i < groups; ++i) {
                rc = group(kWidePerGroup);
                if (rc) return rc;
            }
        }
        ++batch;
        if (first && speculate) {
            if (ev_trav) DGN_HIP(hipEventRecord(ev_trav[3], s));
            DGN_HIP(launch_keep_compact(ca, s, ev ? ev + 4 : nullptr));
            launches += 3 + (g->G > 1);
            compacted = true;
        }
        rc = read_state();
        if (rc) return rc;
        if (!done) compacted = false;      // the speculative pass ran on unfinished masks
        first = false;
    }
    // (a graph that reads nearby and was started wide stays so until its frontiers are far smaller: a wide launch goes many hops,
    // so its frontiers say little about those of the other start, and the way would change with every call)
    const u64 wide_above = (u64)(starts_wide && small_frontier == kNarrowCapNear ? kNarrowCapNear / 4 : small_frontier);
    const bool few_levels = level_launches == 0 && hst->slot[(launch_no - 1) & 1].level <= kNarrowLevels;
    g->wide_hint[hk].store(hst->max_frontier > wide_above && !few_levels ? 1 : 0, std::memory_order_relaxed);
    {
        const int nr = hst->n_runs < kMaxRuns ? hst->n_runs : kMaxRuns;
        bool exact = batch == 1 && used_runs > 0 && hst->n_runs == used_runs;
        for (int r = 0; r < nr; ++r) {
            if (exact && hst->wide_runs[r] != used_len[r]) exact = false;
            g->hint_run_len[hk][r].store(hst->wide_runs[r], std::memory_order_relaxed);
        }
        g->hint_runs[hk].store(nr, std::memory_order_relaxed);
        g->exact_streak[hk].store(exact ? g->exact_streak[hk].load(std::memory_order_relaxed) + 1 : 0,
                                  std::memory_order_relaxed);
    }
    if ((int64_t)hst->slot[(launch_no - 1) & 1].level * kRingLongLevel > g->max_graph_ops && !generic_only && hk == 0)
        g->long_chains.store(1, std::memory_order_relaxed);
    if (recycle && (hst->error & (kErrOverflow | kErrLogFull))) {
        // the log is incomplete; a compaction enqueued ahead may have called it complete
        FillRegion hz[1] = {{S.hdr, sizeof(RecycleHeader)}};
        DGN_HIP(launch_clear(hz, 1, s));
        ++launches;
    }
    if (hst->error & kErrOverflow) {
        // A frontier queue overflowed and dropped entries: restore the fixed point with whole-graph
        // sweeps (each operator re-derives K from its outputs) until one of them changes nothing.
        compacted = false;
        int32_t *changed = &S.state->changed;
        for (;;) {
            FillRegion cz[1] = {{changed, 8}};
            DGN_HIP(launch_clear(cz, 1, s));
            DGN_HIP(launch_fix_sweep(g->v, M, K, flags, changed, grid, s));
            ++launches;
            DGN_HIP(hipMemcpyAsync(pin, S.state, sizeof(TravState), hipMemcpyDeviceToHost, s));
            DGN_HIP(hipStreamSynchronize(s));
            if (!hst->changed) break;
        }
    }
    if (!compacted) {
        if (pq_bytes) {
            FillRegion pq[2] = {{per_query_count, pq_bytes}, {S.pq_part, S.pq_part_bytes}};
            DGN_HIP(launch_clear(pq, 2, s));
            ++launches;
        }
        if (ev_trav) DGN_HIP(hipEventRecord(ev_trav[3], s));
        DGN_HIP(launch_keep_compact(ca, s, ev ? ev + 4 : nullptr));
        launches += 3 + (g->G > 1);
        DGN_HIP(hipStreamSynchronize(s));    // outputs are complete (and the phase events recorded) on return
    }
    if (stats) {
        memset(stats, 0, sizeof(*stats));
        stats->level_trace = user_trace;
        stats->level_trace_cap = user_trace_cap;
        stats->levels = hst->slot[(launch_no - 1) & 1].level;
        if (trace) {
            int64_t nrec = stats->levels < user_trace_cap ? stats->levels : user_trace_cap;
            if (nrec > kTraceLevels) nrec = kTraceLevels;
            if (nrec > 0) {
                DGN_HIP(hipMemcpyAsync(user_trace, S.trace, (size_t)nrec * sizeof(Quad), hipMemcpyDeviceToHost, s));
                DGN_HIP(hipStreamSynchronize(s));
            }
        }
        stats->tensor_visits = (int64_t)hst->tensor_visits;
        stats->max_frontier = (int64_t)hst->max_frontier;
        stats->launches = launches;
        stats->level_launches = level_launches;
        stats->atomic_updates = (int64_t)hst->atomic_updates + num_targets;
        if (recycle) stats->recycled = *reinterpret_cast<const u64 *>(static_cast<const char *>(pin) + sizeof(TravState)) ? 1 : 0;
        if (ev) {
            for (int i = 0; i < 6; ++i) DGN_HIP(hipEventElapsedTime(&stats->phase_ms[i], ev[i], ev[i + 1]));
            DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TOTAL], ev[0], ev[6]));
        } else if (ev_trav) {
            DGN_HIP(hipEventElapsedTime(&stats->phase_ms[DGN_PHASE_TRAVERSE], ev_trav[2], ev_trav[3]));
        }
    }
    return error_bits_to_code(hst->error & ~(kErrOverflow | kErrLogFull));
}

int dgn_prune(const dgn_graph *g, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
              const int32_t *tgt_idx, uint64_t *tensor_mask, uint64_t *op_mask, uint8_t *op_flag, int32_t *kept_ops,
              uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count, void *scratch, size_t scratch_bytes,
              const dgn_options *options, dgn_stats *stats, dgn_stream stream)
{
    return prune_impl(g, num_sets, num_targets, tgt_rowptr, tgt_idx, tensor_mask, op_mask, op_flag, kept_ops, kept_masks,
                      kept_count, per_query_count, scratch, scratch_bytes, options, stats, stream, nullptr, nullptr, num_sets,
                      num_targets);
}

// Removal rule + compaction: K computed from tensor_mask_in (from_tensor_mask), or taken as it stands in op_mask.
// flag_in (or NULL): a byte per operator, 1 exactly where op_mask is not zero (then K is read there only).
static int keep_compact_impl(const dgn_graph *g, const uint64_t *tensor_mask_in, bool from_tensor_mask, uint64_t *op_mask,
                             uint8_t *op_flag, int32_t *kept_ops, uint64_t *kept_masks, int64_t *kept_count,
                             int64_t *per_query_count, void *scratch, size_t scratch_bytes, dgn_stream stream,
                             const uint8_t *flag_in = nullptr)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (!kept_count || !scratch) return DGN_ERR_NULL_PTR;
    if ((g->T > 0 && from_tensor_mask && !tensor_mask_in) || (g->P > 0 && (!op_mask || !kept_ops))) return DGN_ERR_NULL_PTR;
    const PruneScratch S = prune_scratch(scratch, g->P, g->T, g->G, 0);
    if (scratch_bytes < S.bytes) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)scratch | (uintptr_t)tensor_mask_in | (uintptr_t)op_mask | (uintptr_t)kept_masks |
         (uintptr_t)kept_count | (uintptr_t)per_query_count) & 7)
        return DGN_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t pq_bytes = per_query_count ? sizeof(int64_t) * 64 * (size_t)(g->G > 1 ? g->G : 1) : 0;
    FillRegion pq[2] = {{per_query_count, pq_bytes}, {S.pq_part, per_query_count ? S.pq_part_bytes : 0}};
    DGN_HIP(launch_clear(pq, 2, s));
    CompactArgs ca{};
    ca.g = g->v;
    ca.M = reinterpret_cast<const u64 *>(tensor_mask_in);
    ca.K = reinterpret_cast<u64 *>(op_mask);
    ca.op_flag = op_flag;
    ca.kept_ops = kept_ops;
    ca.kept_masks = reinterpret_cast<u64 *>(kept_masks);
    ca.kept_count = kept_count;
    ca.per_query_count = per_query_count;
    ca.opbits = S.opbits;
    ca.block_counts = S.block_counts;
    ca.pq_part = S.pq_part;
    ca.pq_replicas = S.pq_replicas;
    ca.from_tensor_mask = from_tensor_mask;
    ca.flag_in = from_tensor_mask ? nullptr : flag_in;
    DGN_HIP(launch_keep_compact(ca, s));
    return DGN_OK;
}

int dgn_keep_compact(const dgn_graph *g, const uint64_t *tensor_mask_in, uint64_t *op_mask, uint8_t *op_flag,
                     int32_t *kept_ops, uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count,
                     void *scratch, size_t scratch_bytes, dgn_stream stream)
{
    return keep_compact_impl(g, tensor_mask_in, true, op_mask, op_flag, kept_ops, kept_masks, kept_count, per_query_count,
                             scratch, scratch_bytes, stream);
}

// ---- removal rule + compaction for callers that cannot allocate ---------------------------------
// The passes' scratch (kept-operator bitmap, tile counts, replicated per-set counters) lives in an array
// of the code object itself, one copy per device; the host works with its device address, fetched once
// per device, never with the array's name.
constexpr int64_t kStaticMaxOps = (int64_t)1 << 26;
constexpr size_t kStaticBitmapBytes = (size_t)(kStaticMaxOps / 8);
constexpr size_t kStaticCountsBytes = ((size_t)(kStaticMaxOps / kCompactTile + 1) * sizeof(int32_t) + 255) & ~(size_t)255;
constexpr size_t kStaticPqBytes = sizeof(int64_t) * 64 * 64 * kPqStride;
constexpr size_t kStaticScratchBytes = kStaticBitmapBytes + kStaticCountsBytes + kStaticPqBytes;
static __device__ __align__(256) unsigned char static_scratch[kStaticScratchBytes];
constexpr int kStaticMaxDevices = 64;
static std::atomic<void *> g_static_scratch_ptr[kStaticMaxDevices];

// Device address of the current device's copy of the array.
static int static_scratch_address(char **out)
{
    int dev = -1;
    DGN_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kStaticMaxDevices) return DGN_ERR_INVALID_ARG;
    void *p = g_static_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        DGN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(static_scratch)));
        if (!p) return DGN_ERR_INVALID_ARG;
        g_static_scratch_ptr[dev].store(p, std::memory_order_release);   // (two threads racing here fetch the same address)
    }
    *out = static_cast<char *>(p);
    return DGN_OK;
}

int dgn_keep_compact_static_limits(int64_t *max_ops, size_t *static_bytes)
{
    if (max_ops) *max_ops = kStaticMaxOps;
    if (static_bytes) *static_bytes = kStaticScratchBytes;
    return DGN_OK;
}

int dgn_keep_compact_static(const dgn_graph *g, const uint64_t *tensor_mask_in, uint64_t *op_mask, uint8_t *op_flag,
                            int32_t *kept_ops, uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count,
                            dgn_stream stream)
{
    if (!g || !kept_count) return DGN_ERR_NULL_PTR;
    if (g->P > kStaticMaxOps) return DGN_ERR_TOO_LARGE;
    if ((g->T > 0 && !tensor_mask_in) || (g->P > 0 && (!op_mask || !kept_ops))) return DGN_ERR_NULL_PTR;
    if (((uintptr_t)tensor_mask_in | (uintptr_t)op_mask | (uintptr_t)kept_masks | (uintptr_t)kept_count |
         (uintptr_t)per_query_count) & 7)
        return DGN_ERR_INVALID_ARG;
    char *base = nullptr;
    const int rc = static_scratch_address(&base);
    if (rc != DGN_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    CompactArgs ca{};
    ca.g = g->v;
    ca.M = reinterpret_cast<const u64 *>(tensor_mask_in);
    ca.K = reinterpret_cast<u64 *>(op_mask);
    ca.op_flag = op_flag;
    ca.kept_ops = kept_ops;
    ca.kept_masks = reinterpret_cast<u64 *>(kept_masks);
    ca.kept_count = kept_count;
    ca.per_query_count = per_query_count;
    ca.opbits = reinterpret_cast<u64 *>(base);
    ca.block_counts = reinterpret_cast<int32_t *>(base + kStaticBitmapBytes);
    // replicated per-set counters exactly as dgn_keep_compact lays them out: only with few graphs
    ca.pq_replicas = 1;
    while (ca.pq_replicas * 2 * (int64_t)g->G <= 64) ca.pq_replicas *= 2;
    const size_t pq_part_bytes = ca.pq_replicas > 1 ? sizeof(int64_t) * 64 * (size_t)g->G * ca.pq_replicas * kPqStride : 0;
    ca.pq_part = ca.pq_replicas > 1 ? reinterpret_cast<int64_t *>(base + kStaticBitmapBytes + kStaticCountsBytes) : nullptr;
    ca.from_tensor_mask = true;
    // the array keeps what the last call left: the counters must start at zero (a fill kernel, not a memset,
    // so that the call may be captured into a graph)
    const size_t pq_bytes = per_query_count ? sizeof(int64_t) * 64 * (size_t)(g->G > 1 ? g->G : 1) : 0;
    FillRegion pq[2] = {{per_query_count, pq_bytes}, {ca.pq_part, per_query_count ? pq_part_bytes : 0}};
    DGN_HIP(launch_clear(pq, 2, s));
    DGN_HIP(launch_keep_compact(ca, s));
    return DGN_OK;
}

int dgn_prune_words(const dgn_graph *g, int64_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
                    const int32_t *tgt_idx, uint64_t *tensor_mask, uint64_t *op_mask, uint8_t *op_flag, int32_t *kept_ops,
                    uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count, void *scratch,
                    size_t scratch_bytes, const dgn_options *options, dgn_stats *stats, dgn_stream stream)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (num_sets < 1 || num_sets > kMaxCount) return DGN_ERR_TOO_MANY_SETS;
    if (g->G > 1) return DGN_ERR_INVALID_ARG;        // a packed batch already numbers its sets graph by graph
    if (!tgt_rowptr) return DGN_ERR_NULL_PTR;
    const int64_t words = (num_sets + DGN_MAX_SETS - 1) / DGN_MAX_SETS;
    const size_t P = (size_t)g->P, T = (size_t)g->T;
    dgn_options per_word{};
    if (options) per_word = *options;
    if (words > 1) per_word.recycle = 0;             // one scratch buffer serves every word: its log covers the last only
    if (options) options = &per_word;
    dgn_stats total{};
    if (stats) total = *stats;
    total.levels = total.tensor_visits = total.launches = total.level_launches = 0;
    total.max_frontier = 0;
    // Graphs that the ring sweep takes: a workgroup per word, as many words at once as have room in the scratch buffer for
    // what the sweep leaves for the compaction (behind the log, nothing else is in use then).
    PruneScratch S{};
    int ring = 0;
    int64_t at_once = 1;
    if (words > 1) {
        const int rc = check_prune(g, DGN_MAX_SETS, num_targets, tgt_rowptr, tgt_idx, tensor_mask, op_mask, kept_ops, kept_masks,
                                   kept_count, per_query_count, scratch, scratch_bytes, options, &S);
        if (rc) return rc;
        if (ring_waves(g, options, stats, words)) {
            at_once = words_scratch(S, scratch, g->P, words);
            if (at_once > 1) ring = ring_waves(g, options, stats, at_once);
            if (!ring) at_once = 1;
        }
    }
    for (int64_t w = 0; w < words; w += at_once) {
        const int64_t left = num_sets - w * DGN_MAX_SETS;
        const int64_t n_words = words - w < at_once ? words - w : at_once;
        const int32_t q = (int32_t)(left < n_words * DGN_MAX_SETS ? left : n_words * DGN_MAX_SETS);
        // the sets of this word own entries [tgt_rowptr[64w], tgt_rowptr[64w + q]) of tgt_idx: the row
        // pointers hold absolute positions, so the slice is passed as it is and the seed step skips
        // every entry that lies outside it (several words at once: so does every word's workgroup)
        dgn_stats one{};
        if (stats) one = *stats;
        uint64_t *M = tensor_mask ? tensor_mask + w * T : nullptr, *K = op_mask ? op_mask + w * P : nullptr;
        uint64_t *masks = kept_masks ? kept_masks + w * P : nullptr;
        uint8_t *flag = op_flag ? op_flag + w * P : nullptr;
        int32_t *kept = kept_ops ? kept_ops + w * P : nullptr;
        int64_t *count = kept_count ? kept_count + w : nullptr, *pq = per_query_count ? per_query_count + w * 64 : nullptr;
        const int rc = ring ? ring_prune(g, ring, n_words, q, num_targets, tgt_rowptr + w * DGN_MAX_SETS, tgt_idx,
                                         reinterpret_cast<u64 *>(M), reinterpret_cast<u64 *>(K), flag, kept,
                                         reinterpret_cast<u64 *>(masks), count, pq, S, options, stats ? &one : nullptr,
                                         static_cast<hipStream_t>(stream), nullptr, nullptr)
                            : prune_impl(g, q, num_targets, tgt_rowptr + w * DGN_MAX_SETS, tgt_idx, M, K, flag, kept, masks,
                                         count, pq, scratch, scratch_bytes, options, stats ? &one : nullptr, stream,
                                         nullptr, nullptr, words > 1 ? DGN_MAX_SETS : q, num_targets / words);
        if (rc != DGN_OK) return rc;
        if (stats) {
            total.levels += one.levels;
            total.tensor_visits += one.tensor_visits;
            total.launches += one.launches;
            total.level_launches += one.level_launches;
            if (one.max_frontier > total.max_frontier) total.max_frontier = one.max_frontier;
            for (int i = 0; i < 8; ++i) total.phase_ms[i] = (w ? total.phase_ms[i] : 0.0f) + one.phase_ms[i];
        }
    }
    if (stats) *stats = total;
    return DGN_OK;
}

// ---- Backward Prune: scratch = [prune scratch][B: 8T][K of stage one: 8P][its kept list: 4P][small] ----
struct BackwardScratch {
    size_t prune_bytes;
    u64 *B, *KB;
    int32_t *kept, *tgt_rowptr, *flags;
    int64_t *kept_count;
    void *links;            // the lists of the forward stage: in the first stage's queues, which are free by then, or, where
                            // those are smaller, behind the rest
    size_t bytes;
};

static BackwardScratch backward_scratch(void *mem, int64_t P, int64_t T, int64_t Ein, int32_t G)
{
    BackwardScratch b{};
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    b.prune_bytes = up(prune_scratch(nullptr, P, T, G, 0).bytes);
    char *p = static_cast<char *>(mem) + b.prune_bytes;
    b.B = reinterpret_cast<u64 *>(p); p += up((size_t)(T > 0 ? T : 1) * 8);
    b.KB = reinterpret_cast<u64 *>(p); p += up((size_t)(P > 0 ? P : 1) * 8);
    b.kept = reinterpret_cast<int32_t *>(p); p += up((size_t)(P > 0 ? P : 1) * 4);
    b.tgt_rowptr = reinterpret_cast<int32_t *>(p); p += 512;
    b.kept_count = reinterpret_cast<int64_t *>(p); p += up(sizeof(int64_t) * (size_t)(G > 1 ? G + 2 : 1));
    b.flags = reinterpret_cast<int32_t *>(p); p += 256;
    const PruneScratch S = prune_scratch(mem, P, T, G, 0);
    size_t link_bytes = 0;
    (void)backward_links(nullptr, P, Ein, &link_bytes);
    const bool inside = link_bytes <= 2 * align256((size_t)S.qg.S * (size_t)S.qg.seg_cap * sizeof(int32_t));
    b.links = inside ? static_cast<void *>(S.q0) : static_cast<void *>(p);
    b.bytes = (size_t)(p - static_cast<char *>(mem)) + (inside ? 0 : link_bytes);
    return b;
}

int dgn_backward_prune_workspace(const dgn_graph *g, size_t *scratch_bytes)
{
    if (!g || !scratch_bytes) return DGN_ERR_NULL_PTR;
    *scratch_bytes = backward_scratch(nullptr, g->P, g->T, g->Ein, g->G).bytes;
    return DGN_OK;
}

int dgn_backward_prune(const dgn_graph *g, int32_t num_pairs, const int32_t *obj, const int32_t *wrt,
                       uint64_t *tensor_mask, uint64_t *op_mask, uint8_t *op_flag, int32_t *kept_ops,
                       uint64_t *kept_masks, int64_t *kept_count, int64_t *per_query_count, void *scratch,
                       size_t scratch_bytes, const dgn_options *options, dgn_stats *stats, dgn_stream stream)
{
    if (!g) return DGN_ERR_NULL_PTR;
    if (num_pairs < 1 || num_pairs > DGN_MAX_SETS) return DGN_ERR_TOO_MANY_SETS;
    if (g->G > 1) return DGN_ERR_INVALID_ARG;        // pairs are not tied to the graphs of a packed batch
    if (!obj || !wrt || !kept_count || !scratch) return DGN_ERR_NULL_PTR;
    if ((g->T > 0 && !tensor_mask) || (g->P > 0 && (!op_mask || !kept_ops))) return DGN_ERR_NULL_PTR;
    const BackwardScratch S = backward_scratch(scratch, g->P, g->T, g->Ein, g->G);
    if (scratch_bytes < S.bytes) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)scratch | (uintptr_t)tensor_mask | (uintptr_t)op_mask | (uintptr_t)kept_masks |
         (uintptr_t)kept_count | (uintptr_t)per_query_count) & 7)
        return DGN_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    u64 *F = reinterpret_cast<u64 *>(tensor_mask);

    // stage one: what every x_wrt depends on (bit i for pair i), and the operators kept for that
    DGN_HIP(launch_pair_rows(num_pairs, S.tgt_rowptr, s));
    dgn_options o1{};
    if (options) o1 = *options;
    o1.profile = 0;
    o1.incremental = 0;                              // stage one starts from nothing, in scratch memory
    // The marked masks F (the caller's tensor_mask) and the final K (its op_mask) are non-zero only inside stage
    // one's coloured set and kept list, so stage one zeroes them along with its own M and K: everything, or, when
    // the caller recycles the buffers, what the previous call's log and kept list name.
    // Stage one keeps its flag bytes (1 for every operator of its kept list) in the caller's op_flag when that can take
    // them, else in its scratch; the final removal rule turns them into the flags of the result, which spares the
    // last count pass the read of all of K.
    int rc = prune_impl(g, num_pairs, num_pairs, S.tgt_rowptr, wrt, reinterpret_cast<uint64_t *>(S.B),
                        reinterpret_cast<uint64_t *>(S.KB), op_flag, S.kept, nullptr, S.kept_count, nullptr, scratch,
                        S.prune_bytes, &o1, stats, stream, tensor_mask, op_mask, num_pairs, num_pairs);
    if (rc != DGN_OK) return rc;
    uint8_t *stage_flags = nullptr;
    if (!o1.recompute_keep)
        stage_flags = (op_flag && ((uintptr_t)op_flag & 7) == 0 && g->P % 8 == 0)
                          ? op_flag : prune_scratch(scratch, g->P, g->T, g->G, o1.max_queue_entries, true).flagbuf;

    // stage two: forwards from every x_obj, inside the coloured set of stage one
    size_t link_bytes = 0;
    const BackwardLinks L = backward_links(S.links, g->P, g->Ein, &link_bytes);
    DGN_HIP(launch_link_kept(g->v, S.kept, S.kept_count, S.KB, S.B, F, obj, wrt, num_pairs, L, S.flags, g->num_cus, s));
    void *pin = nullptr;
    rc = pinned_buffer(&pin);
    if (rc != DGN_OK) return rc;
    int32_t *host_flags = static_cast<int32_t *>(pin);
    const int grid = g->num_cus * 8;
    // Passes in batches, flags[2 + i] = "pass i of the batch added something", read back after each batch (a read-back
    // idles the GPU for about as long as half a pass takes).  The first batch is as long as the previous call's whole
    // run of passes, the following ones three passes each.
    int64_t passes = 0;
    int batch = g->backward_passes.load(std::memory_order_relaxed) + 1;      // (how far a pass gets varies a little)
    batch = batch < 3 ? 3 : batch > kBackwardMaxBatch ? kBackwardMaxBatch : batch;
    for (;;) {
        FillRegion again[1] = {{S.flags + 2, sizeof(int32_t) * (size_t)kBackwardMaxBatch}};
        if (passes) DGN_HIP(launch_clear(again, 1, s));
        for (int i = 0; i < batch; ++i)
            DGN_HIP(launch_forward_pass(g->v, S.kept_count, S.KB, L, S.flags + 2 + i, g->num_cus, s));
        DGN_HIP(hipMemcpyAsync(host_flags, S.flags, 256, hipMemcpyDeviceToHost, s));
        DGN_HIP(hipStreamSynchronize(s));
        if (host_flags[0] & kErrIdRange) return DGN_ERR_ID_OUT_OF_RANGE;
        int quiet = 0;                               // the first pass of the batch that changed nothing
        while (quiet < batch && host_flags[2 + quiet] != 0) ++quiet;
        if (quiet < batch) {
            g->backward_passes.store((int)(passes + quiet + 1), std::memory_order_relaxed);
            passes += batch;
            break;
        }
        passes += batch;
        batch = 3;
    }
    if (stats) stats->reserved = (int32_t)passes;

    // Removal rule and ordered compaction on the marked set.  A marked tensor lies in stage one's coloured set,
    // so only operators of stage one's kept list can have a marked output: K is cleared and written for those.
    DGN_HIP(launch_write_marks(g->v, g->multi_producer, S.kept, S.kept_count, L.FO, S.B, F, reinterpret_cast<u64 *>(op_mask),
                               stage_flags, grid, s));
    if (g->multi_producer)
        DGN_HIP(launch_keep_from_list(g->v, S.kept, S.kept_count, F, reinterpret_cast<u64 *>(op_mask), stage_flags, grid, s));
    return keep_compact_impl(g, tensor_mask, false, op_mask, op_flag, kept_ops, kept_masks, kept_count, per_query_count,
                             scratch, S.prune_bytes, stream, stage_flags);
}

int dgn_ignore_mask(const dgn_graph *g, const uint64_t *tensor_mask, const int32_t *kept_ops, const uint64_t *kept_masks,
                    const int64_t *kept_count, uint64_t *ignore_mask, int64_t *ignore_count, dgn_stream stream)
{
    if (!g || !kept_count) return DGN_ERR_NULL_PTR;
    if (g->T > 0 && (!tensor_mask || !ignore_mask)) return DGN_ERR_NULL_PTR;
    if (g->P > 0 && (!kept_ops || !kept_masks)) return DGN_ERR_NULL_PTR;
    if (((uintptr_t)tensor_mask | (uintptr_t)kept_masks | (uintptr_t)kept_count | (uintptr_t)ignore_mask |
         (uintptr_t)ignore_count) & 7)
        return DGN_ERR_INVALID_ARG;
    DGN_HIP(launch_ignore_mask(g->v, g->multi_producer, kept_ops, reinterpret_cast<const u64 *>(kept_masks), kept_count,
                               reinterpret_cast<const u64 *>(tensor_mask), reinterpret_cast<u64 *>(ignore_mask),
                               ignore_count, g->num_cus * 2, static_cast<hipStream_t>(stream)));
    return DGN_OK;
}

constexpr int kSetListBlocks = 2048;     // no graph handle here to ask for the number of compute units

int dgn_per_set_lists_workspace(int64_t num_kept, size_t *scratch_bytes)
{
    if (!scratch_bytes) return DGN_ERR_NULL_PTR;
    if (num_kept < 0) return DGN_ERR_INVALID_ARG;
    if (num_kept > kMaxCount / 64) return DGN_ERR_TOO_LARGE;
    *scratch_bytes = set_lists_scratch_bytes(num_kept);
    return DGN_OK;
}

int dgn_per_set_lists(const int32_t *kept_ops, const uint64_t *kept_masks, int64_t num_kept, int64_t *set_rowptr,
                      int32_t *set_ops, int64_t set_ops_capacity, void *scratch, size_t scratch_bytes, dgn_stream stream)
{
    if (num_kept < 0 || set_ops_capacity < 0) return DGN_ERR_INVALID_ARG;
    if (num_kept > kMaxCount / 64) return DGN_ERR_TOO_LARGE;      // slots are counted in int32
    if (!set_rowptr || !scratch) return DGN_ERR_NULL_PTR;
    if (num_kept > 0 && (!kept_ops || !kept_masks)) return DGN_ERR_NULL_PTR;
    if (set_ops_capacity > 0 && !set_ops) return DGN_ERR_NULL_PTR;
    if (scratch_bytes < set_lists_scratch_bytes(num_kept)) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)kept_masks | (uintptr_t)set_rowptr | (uintptr_t)scratch) & 7) return DGN_ERR_INVALID_ARG;
    DGN_HIP(launch_set_lists(kept_ops, reinterpret_cast<const u64 *>(kept_masks), num_kept, set_rowptr, set_ops,
                             set_ops_capacity, scratch, kSetListBlocks, static_cast<hipStream_t>(stream)));
    return DGN_OK;
}

int dgn_target_digest_workspace(size_t *scratch_bytes)
{
    if (!scratch_bytes) return DGN_ERR_NULL_PTR;
    *scratch_bytes = digest_scratch_bytes();
    return DGN_OK;
}

int dgn_target_digest(const dgn_graph *g, int32_t num_sets, int64_t num_targets, const int32_t *tgt_rowptr,
                      const int32_t *tgt_idx, uint64_t *digest_out, void *scratch, size_t scratch_bytes, dgn_stream stream)
{
    if (!g || !tgt_rowptr || !digest_out || !scratch) return DGN_ERR_NULL_PTR;
    if (num_sets < 1 || num_sets > DGN_MAX_SETS) return DGN_ERR_TOO_MANY_SETS;
    if (num_targets < 0) return DGN_ERR_INVALID_ARG;
    if (num_targets > kMaxCount) return DGN_ERR_TOO_LARGE;
    if (num_targets > 0 && !tgt_idx) return DGN_ERR_NULL_PTR;
    if (scratch_bytes < digest_scratch_bytes()) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if ((uintptr_t)scratch & 7) return DGN_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    u64 *dev = nullptr;
    DGN_HIP(launch_target_digest(num_sets, (int64_t)num_sets * g->G, tgt_rowptr, num_targets, tgt_idx, scratch, &dev, s));
    void *pin = nullptr;
    const int rc = pinned_buffer(&pin);
    if (rc != DGN_OK) return rc;
    DGN_HIP(hipMemcpyAsync(pin, dev, 2 * sizeof(u64), hipMemcpyDeviceToHost, s));
    DGN_HIP(hipStreamSynchronize(s));
    digest_out[0] = static_cast<const u64 *>(pin)[0];
    digest_out[1] = static_cast<const u64 *>(pin)[1];
    return DGN_OK;
}

int dgn_inplace_workspace(const dgn_graph *g, size_t *scratch_bytes)
{
    if (!g || !scratch_bytes) return DGN_ERR_NULL_PTR;
    *scratch_bytes = inplace_scratch_bytes(g->T);
    return DGN_OK;
}

static int inplace_impl(const dgn_graph *g, const uint64_t *op_mask, uint64_t select, const int32_t *kept_ops,
                        const int64_t *kept_count, int32_t *rename, int64_t *renamed_count, void *scratch,
                        size_t scratch_bytes, int32_t *rounds_out, dgn_stream stream)
{
    if (!g || !scratch) return DGN_ERR_NULL_PTR;
    if ((g->P > 0 && !op_mask) || (g->T > 0 && !rename)) return DGN_ERR_NULL_PTR;
    if (scratch_bytes < inplace_scratch_bytes(g->T)) return DGN_ERR_WORKSPACE_TOO_SMALL;
    if (((uintptr_t)scratch | (uintptr_t)op_mask | (uintptr_t)renamed_count) & 7) return DGN_ERR_INVALID_ARG;
    if ((uintptr_t)rename & 3) return DGN_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const InplaceBuffers B = inplace_buffers(scratch, g->T);
    const int grid = g->num_cus * 8;
    DGN_HIP(launch_inplace_setup(g->v, reinterpret_cast<const u64 *>(op_mask), select, kept_ops, kept_count, rename,
                                 renamed_count, B, g->meet, grid, s));
    void *pin = nullptr;
    int rc = pinned_buffer(&pin);
    if (rc != DGN_OK) return rc;
    int round = 0;
    for (;;) {                                       // four rounds per read-back of the "still alive" word
        for (int i = 0; i < 4 && round < kInplaceMaxRounds; ++i, ++round)
            DGN_HIP(launch_inplace_round(round, rename, renamed_count, B, grid, s));
        DGN_HIP(hipMemcpyAsync(pin, B.counters + round, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        DGN_HIP(hipStreamSynchronize(s));
        if (*static_cast<int32_t *>(pin) == 0 || round >= kInplaceMaxRounds) break;
    }
    if (rounds_out) *rounds_out = round;
    return DGN_OK;
}

int dgn_inplace(const dgn_graph *g, const uint64_t *op_mask, uint64_t select, int32_t *rename, int64_t *renamed_count,
                void *scratch, size_t scratch_bytes, int32_t *rounds_out, dgn_stream stream)
{
    return inplace_impl(g, op_mask, select, nullptr, nullptr, rename, renamed_count, scratch, scratch_bytes, rounds_out,
                        stream);
}

int dgn_inplace_kept(const dgn_graph *g, const uint64_t *op_mask, uint64_t select, const int32_t *kept_ops,
                     const int64_t *kept_count, int32_t *rename, int64_t *renamed_count, void *scratch,
                     size_t scratch_bytes, int32_t *rounds_out, dgn_stream stream)
{
    if (g && g->P > 0 && (!kept_ops || !kept_count)) return DGN_ERR_NULL_PTR;
    if ((uintptr_t)kept_count & 7) return DGN_ERR_INVALID_ARG;
    return inplace_impl(g, op_mask, select, kept_ops, kept_count, rename, renamed_count, scratch, scratch_bytes,
                        rounds_out, stream);
}

}  // extern "C"
