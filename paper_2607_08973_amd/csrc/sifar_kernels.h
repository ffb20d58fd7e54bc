// Internal interface between the host runtime (api.cpp) and the gfx950
// kernels (kernels.hip). Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sifar {

constexpr int kLanes = 64;                 // wavefront width on CDNA
constexpr int kVec = 8;                    // bf16 elements per 16-byte load
constexpr int kChunk = kLanes * kVec;      // elements per chunk: one wave, one load per rank per lane
constexpr int kMaxRanks = 8;
constexpr int kMaxWavesPerGroup = 16;
constexpr int kStepConsumers = 4;           // consumer waves of a one-launch step's chunk when split
constexpr int kSplitChunks = 256;           // most chunks of a step that splits them
constexpr int kExchPlanes = 4;              // epoch-indexed planes of the epilogue exchange
// Least bound on the exchange wait of a one-launch step whose launches, one per
// all-reduce, would not wait between workgroups (0.5 s or more of polls).
constexpr uint32_t kStepSpins = 1u << 20;

// x % d for a divisor fixed per launch, by a multiply-high instead of a
// division sequence (Granlund and Montgomery, "Division by invariant integers
// using multiplication", 1994, unsigned case): with l = ceil(log2 d) and
// m = floor(2^32 (2^l - d) / d) + 1, the quotient of a 32-bit x is
// (t + ((x - t) >> min(l, 1))) >> max(l - 1, 0), t = the high word of m * x.
struct DivU32 {
    uint32_t m, sh1, sh2, d;
};

__host__ __device__ inline DivU32 make_div(uint32_t d) {
    uint32_t l = 0;
    while (l < 32 && (uint64_t{1} << l) < d) ++l;
    DivU32 v;
    v.m = static_cast<uint32_t>(((uint64_t{1} << 32) * ((uint64_t{1} << l) - d)) / d + 1);
    v.sh1 = l < 1 ? l : 1;
    v.sh2 = l > 1 ? l - 1 : 0;
    v.d = d;
    return v;
}

__host__ __device__ inline uint32_t mod_u32(uint32_t x, const DivU32 &v) {
    const uint32_t t = static_cast<uint32_t>((static_cast<uint64_t>(v.m) * x) >> 32);
    const uint32_t q = (t + ((x - t) >> v.sh1)) >> v.sh2;
    return x - q * v.d;
}

// Token rows of a persistent plain step's planes: a plane of `tokens` rows of
// `segs` one-wave workgroups, with rows of idle workgroups added until it is a
// multiple of the 8 XCDs. Workgroups are dealt to the XCDs round robin, plane
// 1 after plane 0, so a chunk's consumer and producer then share an XCD
// whatever the shape. Without the added rows 45 chunks (N = 8, 5 tokens x
// 4608) put every pair on two XCDs, which pays a release fence per epoch:
// 162 us a 64-all-reduce step, 47 with them. (A macro, so that a test can build
// the library with 1 and still run the cross-XCD handoffs.)
#ifndef SIFAR_PLANE_ALIGN
#define SIFAR_PLANE_ALIGN 8
#endif
inline int64_t plane_rows(int64_t tokens, int64_t segs) {
    while (tokens * segs % SIFAR_PLANE_ALIGN != 0) ++tokens;
    return tokens;
}

// Device-resident state shared by all kernels of a handle.
struct DevState {
    uint32_t epoch_base;   // graph nodes compute g = epoch_base + node offset
    uint32_t zero;         // always 0: eager launches pass g as the offset
    uint32_t err[4];       // kind, epoch, chunk, attempts (first error wins)
    uint32_t chain_done;   // waves of the running persistent step that have finished
};

// Geometry common to the producer and the reduction.
struct Geometry {
    int32_t nranks;
    int32_t tokens;
    int32_t hidden;
    int32_t segs;          // chunks per token = ceil(hidden / kChunk)
    int32_t w_max;         // max_tokens * segs: stride of the stamp and log rows
    uint64_t slot_elems;   // elements between consecutive slots
};

// Where the epoch of a launch comes from: g = *base + off. The slot parity is
// frozen at launch (graph capture) time -- g & 1 with dual buffering (the host
// keeps *base even for graphs), 0 with a single buffer.
struct EpochRef {
    const uint32_t *base;
    uint32_t off;
    uint32_t parity;
};

struct ProduceArgs {
    Geometry geo;
    EpochRef ep;
    uint16_t *slots;             // [N][2][slot_elems]
    uint32_t *stamps;            // [2][w_max][N]
    const uint32_t *consumed;    // [2][w_max]: last epoch whose reduction finished the chunk
    uint32_t *produced;          // [2][w_max]: last epoch written into the chunk's slots
    const uint16_t *src;         // entry e, rank r: src + e*entry_stride + r*rank_stride
    int64_t entry_stride;
    int64_t rank_stride;
    int32_t entries;             // epoch g uses entry (g - 1) % entries
    DivU32 entries_div;          // make_div(entries)
    const uint16_t *inject;      // [inject_entries] late | withheld << 8, or null
    int32_t inject_entries;
    DivU32 inject_div;           // make_div(inject_entries), or make_div(1) without a table
    uint16_t *stage;             // [N][2][slot_elems], or null: with deterministic injection a
                                 // late rank's payload is written here, not into its slot, and
                                 // the reduction moves it into the slot when the rank catches up
    uint32_t *err;
};

struct ReduceArgs {
    Geometry geo;
    EpochRef ep;
    uint16_t *slots;             // written only when a late rank catches up (deterministic injection)
    uint32_t *stamps;
    uint32_t *consumed;
    uint32_t *log;               // [log_epochs][w_max]
    uint32_t *stamp_log;         // [log_epochs][w_max][2][N]: the raw stamps of the chunk's first
                                 // and last validation (per-epoch launches: may be null)
    int32_t log_epochs;
    DivU32 log_div;              // make_div(log_epochs)
    uint32_t max_attempts;
    uint32_t forced_retries;
    uint32_t spin_limit;
    const uint16_t *inject;
    int32_t inject_entries;
    DivU32 inject_div;
    const uint16_t *stage;       // late ranks' payload (ProduceArgs::stage), or null
    uint16_t *out;               // plain: [tokens][hidden]
    uint16_t *residual;          // epilogue: [tokens][hidden], in place
    const uint16_t *weight;      // [hidden]
    uint16_t *y;                 // [tokens][hidden]
    uint64_t *exch;              // [kExchPlanes][words]: token t's word of group q at
                                 // t * groups_per_token + q: (epoch << 32) | partial bits;
                                 // per-launch epilogues use planes g & 1, one-launch and
                                 // persistent steps g mod kExchPlanes
    int32_t groups_per_token;
    int32_t exch_parity_stride;  // words per exchange plane
    float eps;
    uint32_t *err;
};

// One launch running a whole decode step: consumer waves (plane 0) reduce the
// L epochs one after another while producer waves (plane 1) play the peers,
// concurrently, synchronised only through stamps and consumed/produced words.
struct ChainArgs {
    ReduceArgs r;                // r.out / r.y point at ring entry 0
    ProduceArgs p;
    int32_t reduces;             // L
    uint64_t ring_stride;        // elements between ring entries
    uint32_t late_delay;         // injected late stamps land after this many sleeps
    uint32_t *epoch_base;        // advanced by `advance` by the last wave to finish
    uint32_t advance;
    uint32_t *done;              // arrival counter of the step's waves (left at 0)
    uint32_t parity_mask;        // 1: dual buffering (parity = epoch & 1); 0: one slot
    uint64_t *place;             // [2][w_max]: plane 0 consumer, plane 1 producer of each
                                 // chunk: (base + 1) << 32 | 0x100 | XCD, written at step start
};

// One all-reduce of one epoch in one launch: what it needs beyond geometry,
// sources, slots and stamps.
struct OnceArgs {
    uint32_t *consumed;          // [2][w_max]
    uint32_t *produced;          // [2][w_max]
    uint32_t *log;               // [w_max]
    uint16_t *out;               // [tokens][hidden]
    uint32_t max_attempts;
    uint32_t *err;
};

enum Mode : int { kSpec = 0, kOrdered = 1, kNone = 2 };

hipError_t launch_produce(const ProduceArgs &a, int waves_per_group, hipStream_t s);
// With `next` non-null the launch also produces the next epoch (fused peers).
hipError_t launch_reduce(const ReduceArgs &a, const ProduceArgs *next, int mode, bool epilogue,
                         int waves_per_group, hipStream_t s);
// Workgroups of the reduction kernel that can be resident at once on the
// current device (0 if unknown).
int max_active_groups(int nranks, int mode, bool epilogue, int waves_per_group);
// Same for the persistent chain kernel's one-wave workgroups; `prefetch` picks
// the plain kernel whose producer loads an epoch's sources ahead (more
// registers, lower occupancy).
int max_active_chain_waves(int nranks, int mode, bool epilogue, bool prefetch);
// Persistent step: grid (segs, plane_rows(tokens, segs), 2), or with the
// epilogue one that puts a token's workgroups on one XCD.
hipError_t launch_chain(const ChainArgs &a, int mode, bool epilogue, bool prefetch, hipStream_t s);
// One-launch steps address the slots at 32-bit offsets from rank 0's.
inline bool step_offsets_fit(int nranks, uint64_t slot_elems) {
    return static_cast<uint64_t>(nranks) * 4u * slot_elems <= 0x7fffffffull;
}
inline bool source_offsets_fit(int nranks, int64_t rank_stride) {
    return rank_stride <= 0x7fffffffll / 2 / nranks;
}
// All-reduce of epoch g in one launch, a two-wave workgroup per chunk.
hipError_t launch_once(const Geometry &geo, uint32_t g, const uint16_t *src, int64_t rank_stride,
                       uint16_t *slots, uint32_t *stamps, const OnceArgs &a, hipStream_t s);
// Per-epoch step in one launch (dual buffers): a workgroup per chunk, of
// `consumers` (1, or without an injection table kStepConsumers) reducing waves
// and one of the peers; how many workgroups with one, and with kStepConsumers,
// can be resident at once.
hipError_t launch_step(const ChainArgs &a, int mode, bool epilogue, int consumers,
                       hipStream_t s);
int max_active_step_groups(int nranks, int mode, bool epilogue);
int max_active_split_step_groups(int nranks, int mode, bool epilogue);
hipError_t launch_advance(uint32_t *epoch_base, uint32_t step, hipStream_t s);
hipError_t launch_set_base(uint32_t *epoch_base, uint32_t value, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, uint32_t value, uint64_t count, hipStream_t s);

}  // namespace sifar
