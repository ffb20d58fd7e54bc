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
    // steps: a written array that overlaps anything else, each pair in turn
    uint64_t steps[2] = {0, 0};
    for (int i = 0; i < 200000; ++i) {
        StepSpans b{};
        b.src.block = draw(1, 8);
        b.src.ranks = draw(1, 3);
        b.src.rank_bytes = b.src.block + draw(0, 30);
        b.src.entries = draw(1, 3);
        b.src.entry_bytes = b.src.ranks * b.src.rank_bytes + draw(0, 30);
        b.src.at = draw(0, 200);
        b.ring = Span{draw(0, 600), draw(1, 24)};
        if (rng() % 2) b.residual = Span{draw(0, 600), draw(1, 8)}, b.weight = Span{draw(0, 600), draw(1, 8)};
        Map m(kBytes * 2, 0);  // bits: 1 source, 2 ring, 4 residual, 8 weight
        for (uint64_t e = 0; e < b.src.entries; ++e)
            for (uint64_t r = 0; r < b.src.ranks; ++r)
                for (uint64_t k = 0; k < b.src.block; ++k)
                    m.at(b.src.at + e * b.src.entry_bytes + r * b.src.rank_bytes + k) |= 1;
        for (uint64_t k = 0; k < b.ring.size; ++k) m.at(b.ring.at + k) |= 2;
        for (uint64_t k = 0; k < b.residual.size; ++k) m.at(b.residual.at + k) |= 4;
        for (uint64_t k = 0; k < b.weight.size; ++k) m.at(b.weight.at + k) |= 8;
        bool want = false;  // a written byte that something else holds too
        for (int x : m) want |= (x & 6) != 0 && (x & (x - 1)) != 0;
        if (step_overlaps(b) != want) return std::printf("FAIL step\n"), 1;
        ++steps[want];
    }
    if (!steps[0] || !steps[1]) return std::printf("FAIL: a kind of step was never drawn\n"), 1;
    if (!met || !raced || !equal) return std::printf("FAIL: a kind of layout was never drawn\n"), 1;
    std::printf("ok %llu\n", (unsigned long long)checked);
    return 0;
}
