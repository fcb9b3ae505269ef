// Host-only check of the library's scratch layouts (compiled and run by test_scratch_layout.py; nothing touches a GPU): the
// regions that one call of the ring sweep writes must lie inside the scratch buffer and must not overlap.  The layout
// functions are internal to api.hip, so this file includes it.
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

int main()
{
    char *base = reinterpret_cast<char *>((uintptr_t)1 << 40);              // (never dereferenced)
    uint8_t *given = reinterpret_cast<uint8_t *>((uintptr_t)1 << 41);
    const int64_t ops[] = {1, 63, 64, 257, 3001, 9000, 16384, 16385, 18501, 20000, 20001, 23999, 25001, 26501, 32768, 65537, 131072};
    const double ratios[] = {0.001, 0.5, 1.0, 1.25, 1.5, 2.0, 3.0};
    long long bad = 0, layouts = 0, chunked = 0;
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
                    }
    printf("%lld layouts, %lld with more words than room, %lld faults\n", layouts, chunked, bad);
    return bad != 0;
}
