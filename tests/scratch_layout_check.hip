// Host-only check of the library's scratch layouts (compiled and run by test_scratch_layout.py; nothing touches a GPU): the
// regions that one call of the ring sweep (in one piece or in segments) or of the sweep by layers writes must lie inside the scratch
// buffer and must not overlap.  The layout functions are internal to api.hip, so this file includes it.
#include "../paper_1707_08265_amd/csrc/api.hip"

#include <stdio.h>
#include <vector>

struct Region { const char *name; uintptr_t at; size_t bytes; };

static int overlaps(const std::vector<Region> &r, uintptr_t lo, uintptr_t hi, const char *what, long long P, long long T, long long words)
{
    int bad = 0;
    for (size_t i = 0; i < r.size(); ++i) {
        if (r[i].at < lo || r[i].at + r[i].bytes > hi) {
            printf("%s P=%lld T=%lld words=%lld: %s leaves the buffer\n", what, P, T, words, r[i].name);
            ++bad;
        }
        for (size_t j = 0; j < i; ++j)
            if (r[i].at < r[j].at + r[j].bytes && r[j].at < r[i].at + r[i].bytes) {
                printf("%s P=%lld T=%lld words=%lld: %s overlaps %s\n", what, P, T, words, r[i].name, r[j].name);
                ++bad;
            }
    }
    return bad;
}

static char *const base = reinterpret_cast<char *>((uintptr_t)1 << 40);     // (never dereferenced)
static uint8_t *const given = reinterpret_cast<uint8_t *>((uintptr_t)1 << 41);

// Graphs of P operators in all that may be swept in segments: the regions of such a call behind those in r.  How many segments, 1: none.
static int segment_regions(std::vector<Region> &r, const PruneScratch &S, int64_t P, int64_t T, int32_t G, int64_t largest, int64_t words,
                           int low, int64_t targets)
{
    dgn_graph g{};
    g.P = P; g.T = T; g.G = G; g.num_cus = 256; g.max_graph_ops = largest; g.ring_reach = kWave; g.ring_low = low;
    g.v.num_ops = (int32_t)P; g.v.num_tensors = (int32_t)T; g.v.num_graphs = G;
    RingArgs a{};
    a.g = g.v; a.words = (int32_t)words; a.low_words = low; a.num_targets = targets;
    const int segs = ring_segments(&g, words, segments_room(S, words), a);
    if (segs < 2) return 1;
    const size_t rows = (size_t)G * segs;
    r.push_back({"M of the boundaries", (uintptr_t)a.b_M, (size_t)T * 8});
    r.push_back({"K of the boundaries", (uintptr_t)a.b_K, (size_t)P * 8});
    r.push_back({"edges", (uintptr_t)a.edge, rows * (size_t)(words + 1) * (size_t)ring_edge_words(a) * 8});
    r.push_back({"own bits", (uintptr_t)a.own_bits, (size_t)ring_bit_words(P, G) * (size_t)words * 8});
    if (G > 1) r.push_back({"kept per segment", (uintptr_t)a.seg_kept, rows * 4});
    return segs;
}

int main()
{
    const int64_t ops[] = {1, 63, 64, 257, 3001, 9000, 16384, 16385, 18501, 20000, 20001, 23999, 25001, 26501, 32768, 65537, 131072};
    const double ratios[] = {0.001, 0.5, 1.0, 1.25, 1.5, 2.0, 3.0};
    long long bad = 0, layouts = 0, chunked = 0, segmented = 0, layered = 0;
    for (int64_t P : ops)
        for (double ratio : ratios)
            for (int64_t entries : {(int64_t)0, (int64_t)1, (int64_t)64})
                for (int64_t words : {(int64_t)1, (int64_t)2, (int64_t)3, (int64_t)100, (int64_t)100000})
                    for (uint8_t *flag : {(uint8_t *)nullptr, given, given + 1}) {
                        const int64_t T = (int64_t)(ratio * (double)P) + 1;
                        PruneScratch S = prune_scratch(base, P, T, 1, entries);
                        const int64_t at_once = words > 1 ? words_scratch(S, base, P, words) : 1;
                        if (at_once < words && words < 100000) ++chunked;
                        const size_t per = (size_t)ring_bit_words(P, 1) * (size_t)at_once;
                        std::vector<Region> r = {{"header", (uintptr_t)S.hdr, 4 * sizeof(RecycleHeader)},
                                                 {"bits", (uintptr_t)S.ring_bits, per * sizeof(u64)},
                                                 {"running counts", (uintptr_t)S.ring_cum, per * sizeof(int32_t)},
                                                 {"records", (uintptr_t)S.ring_graphs, (size_t)at_once * sizeof(int4)}};
                        const uint8_t *flags = ring_flags(S, flag, P);
                        if (flags != flag) r.push_back({"flags", (uintptr_t)flags, (size_t)P});
                        bad += overlaps(r, (uintptr_t)base, (uintptr_t)base + S.bytes, "ring sweep", P, T, words);
                        ++layouts;
                        for (int low : {1, 16, 300}) {
                            std::vector<Region> more = r;
                            if (segment_regions(more, S, P, T, 1, P, at_once, low, 100) < 2) continue;
                            bad += overlaps(more, (uintptr_t)base, (uintptr_t)base + S.bytes, "segments", P, T, words);
                            ++segmented;
                        }
                    }
    for (int32_t G : {2, 8, 63, 64, 96, 250, 600})
        for (int64_t each : {450, 1000, 3001, 20000})
            for (double part : {1.0, 0.6, 0.1})             // operators in all, against all graphs as large as the largest
                for (double ratio : ratios)
                    for (uint8_t *flag : {(uint8_t *)nullptr, given, given + 1}) {
                        const int64_t P = (int64_t)(part * (double)(each * G)) + each, T = (int64_t)(ratio * (double)P) + 16 * G;
                        const PruneScratch S = prune_scratch(base, P, T, G, 0);
                        std::vector<Region> r = {{"header", (uintptr_t)S.hdr, 4 * sizeof(RecycleHeader)},
                                                 {"bits", (uintptr_t)S.ring_bits, (size_t)ring_bit_words(P, G) * sizeof(u64)},
                                                 {"running counts", (uintptr_t)S.ring_cum, (size_t)ring_bit_words(P, G) * sizeof(int32_t)},
                                                 {"records", (uintptr_t)S.ring_graphs, ((size_t)G + 1) * sizeof(int4)}};
                        const uint8_t *flags = ring_flags(S, flag, P);
                        if (flags != flag) r.push_back({"flags", (uintptr_t)flags, (size_t)P});
                        if (segment_regions(r, S, P, T, G, each, 1, 16, 4 * G) < 2) continue;
                        bad += overlaps(r, (uintptr_t)base, (uintptr_t)base + S.bytes, "segments of a batch", P, T, 1);
                        ++segmented;
                    }
    // The sweep by layers, also as a first stage that keeps flag bytes of its own; with small queues it may have no room
    for (int64_t P : {1, 511, 8192, 8193, 16807, 40000, 200001, 1 << 20})
        for (double ratio : ratios)
            for (int64_t entries : {(int64_t)0, (int64_t)1, (int64_t)1 << 20})
                for (bool stage : {false, true})
                    for (uint8_t *flag : {(uint8_t *)nullptr, given, given + 1}) {
                        const int64_t T = (int64_t)(ratio * (double)P) + 1;
                        const PruneScratch S = prune_scratch(base, P, T, 1, entries, stage);
                        BandArgs a{};
                        a.g.num_ops = (int32_t)P;
                        if (reinterpret_cast<const char *>(S.q0) + band_scratch(a, nullptr) > reinterpret_cast<const char *>(S.flagbuf)) continue;
                        const size_t bytes = band_scratch(a, S.q0);
                        std::vector<Region> r = {{"header", (uintptr_t)S.hdr, 4 * sizeof(RecycleHeader)},
                                                 {"state", (uintptr_t)S.state, 256 + sizeof(TravCounters)},
                                                 {"operators", (uintptr_t)a.entry, (size_t)P * 12},
                                                 {"steps", (uintptr_t)a.steps, (uintptr_t)a.segs - (uintptr_t)a.steps},
                                                 {"segments", (uintptr_t)a.segs, (uintptr_t)S.q0 + bytes - (uintptr_t)a.segs},
                                                 {"bits", (uintptr_t)S.opbits, S.opbits_bytes},
                                                 {"counts", (uintptr_t)S.block_counts, (size_t)((P + kCompactTile - 1) / kCompactTile + 1) * 4},
                                                 {"per-set counts", (uintptr_t)S.pq_part, S.pq_part_bytes}};
                        const uint8_t *flags = stage ? ring_flags(S, flag, P) : flag;
                        if (flags != flag) r.push_back({"flags", (uintptr_t)flags, S.db_bytes});
                        bad += overlaps(r, (uintptr_t)base, (uintptr_t)base + S.bytes, "sweep by layers", P, T, 1);
                        ++layered;
                    }
    printf("%lld layouts, %lld with more words than room, %lld in segments, %lld by layers, %lld faults\n", layouts, chunked, segmented, layered, bad);
    if (segmented < 1000 || layered < 100) return 2;
    return bad != 0;
}
