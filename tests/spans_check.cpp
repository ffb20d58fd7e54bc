// Host-side check of the buffer-overlap rules (spans.h) against a byte map:
// random small layouts, every rule compared with the sets of bytes it speaks of.
// Built and run by tests/test_spans.py on the CPU (no GPU call).
#include <cstdio>
#include <random>
#include <vector>

#include "spans.h"

using namespace sifar;

namespace {

constexpr uint64_t kBytes = 640;
typedef std::vector<int> Map;  // per byte: 0, or 1 + the index of the block that holds it

bool meets(const Map &m, const Span &s) {
    for (uint64_t i = s.at; i < s.at + s.size; ++i)
        if (m[i]) return true;
    return false;
}

}  // namespace

int main() {
    std::mt19937_64 rng(260708973);
    auto draw = [&](uint64_t lo, uint64_t hi) { return lo + rng() % (hi - lo + 1); };
    uint64_t checked = 0, met = 0, raced = 0, equal = 0;
    while (checked < 400000) {
        Blocks b{};
        b.block = draw(1, 12);
        b.ranks = draw(1, 4);
        b.rank_bytes = b.block + (rng() % 2 ? draw(0, 9) : 0);
        b.entries = draw(1, 5);
        b.entry_bytes = b.ranks * b.rank_bytes + (rng() % 2 ? draw(0, 15) : 0);
        if (b.entries == 1 && rng() % 2) b.entry_bytes = draw(0, 9);  // unused with one entry
        b.at = draw(0, 40);
        Map m(kBytes, 0);
        for (uint64_t e = 0; e < b.entries; ++e)
            for (uint64_t r = 0; r < b.ranks; ++r)
                for (uint64_t i = 0; i < b.block; ++i)
                    m.at(b.at + (b.entries > 1 ? e * b.entry_bytes : 0) + r * b.rank_bytes + i) = 1;
        const Span s{draw(0, 600), draw(0, 30)};
        const bool want = meets(m, s);
        if (overlap(b, s) != want) {
            std::printf("FAIL overlap: blocks at %llu entries %llu x %llu ranks %llu x %llu block "
                        "%llu, span %llu + %llu: want %d\n",
                        (unsigned long long)b.at, (unsigned long long)b.entries,
                        (unsigned long long)b.entry_bytes, (unsigned long long)b.ranks,
                        (unsigned long long)b.rank_bytes, (unsigned long long)b.block,
                        (unsigned long long)s.at, (unsigned long long)s.size, want);
            return 1;
        }
        met += want;
        const Span t{draw(0, 600), draw(0, 30)};
        Map ms(kBytes, 0);
        for (uint64_t i = s.at; i < s.at + s.size; ++i) ms[i] = 1;
        if (overlap(s, t) != meets(ms, t)) return std::printf("FAIL span\n"), 1;

        // one launch: byte i of `out` is written while byte i of every block may
        // not have been read by another chunk yet. A chunk is one byte here: the
        // write of out[i] may only touch blocks' byte i.
        b.entries = 1;
        const Span out{rng() % 3 ? draw(0, 80) : b.at + draw(0, b.ranks - 1) * b.rank_bytes, b.block};
        bool race = false;
        for (uint64_t i = 0; i < out.size; ++i)
            for (uint64_t r = 0; r < b.ranks; ++r)
                for (uint64_t j = 0; j < b.block; ++j)
                    if (out.at + i == b.at + r * b.rank_bytes + j && i != j) race = true;
        if (chunks_race(b, out) != race) return std::printf("FAIL race\n"), 1;
        raced += race;
        equal += !race && overlap(b, out);
        ++checked;
    }
    if (!met || !raced || !equal) return std::printf("FAIL: a kind of layout was never drawn\n"), 1;
    std::printf("ok %llu\n", (unsigned long long)checked);
    return 0;
}
