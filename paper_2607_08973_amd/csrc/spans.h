// Which buffers of a call overlap: host-side rules that keep an all-reduce off
// the one-launch kernels when its writes could meet another chunk's reads.
// Plain C++ (bytes and addresses only).
#pragma once
#include <cstdint>

namespace sifar {

// Bytes [at, at + size).
struct Span {
    uint64_t at = 0, size = 0;
};

inline bool overlap(const Span &a, const Span &b) {
    return a.size != 0 && b.size != 0 && a.at < b.at + b.size && b.at < a.at + a.size;
}

// Source blocks: `entries` x `ranks` blocks of `block` bytes, entries and ranks
// at least `block` bytes apart.
struct Blocks {
    uint64_t at = 0;
    uint64_t entries = 1, entry_bytes = 0;
    uint64_t ranks = 1, rank_bytes = 0;
    uint64_t block = 0;
};

// Does a block overlap `s`? Blocks may leave gaps between them that `s` lies in.
inline bool overlap(const Blocks &b, const Span &s) {
    for (uint64_t r = 0; r < b.ranks; ++r) {
        const uint64_t at = b.at + r * b.rank_bytes;  // of entry 0
        if (b.entries <= 1 || b.entry_bytes == 0) {
            if (overlap(Span{at, b.block}, s)) return true;
            continue;
        }
        // the last entry whose block starts before s ends: earlier ones end earlier
        const uint64_t end = s.at + s.size;
        if (s.size == 0 || end <= at) continue;
        uint64_t e = (end - 1 - at) / b.entry_bytes;
        if (e >= b.entries) e = b.entries - 1;
        if (overlap(Span{at + e * b.entry_bytes, b.block}, s)) return true;
    }
    return false;
}

// One all-reduce in one launch: every chunk reads its part of each rank's block,
// then writes its part of `out`, and chunks wait for nothing. Safe where `out`
// is clear of the blocks, or exactly one of them (a chunk then overwrites what
// only it reads). Otherwise the reads have to be a launch of their own.
inline bool chunks_race(const Blocks &src, const Span &out) {
    for (uint64_t r = 0; r < src.ranks; ++r) {
        const Span rank{src.at + r * src.rank_bytes, src.block};
        if (overlap(rank, out) && rank.at != out.at) return true;
    }
    return false;
}

// What a decode step is bound to: it reads the sources and the weight, writes the
// ring of outputs and updates the residual.
struct StepSpans {
    Blocks src;
    Span ring, residual, weight;
};

// A step in one launch: chunks run their whole step free of each other, sources
// are read a phase ahead, and residual and weight stay in registers. Safe where
// nothing the step writes overlaps anything else it touches; otherwise its
// phases have to be launches.
inline bool step_overlaps(const StepSpans &b) {
    return overlap(b.src, b.ring) || overlap(b.src, b.residual) || overlap(b.ring, b.residual) ||
           overlap(b.ring, b.weight) || overlap(b.residual, b.weight);
}

}  // namespace sifar
