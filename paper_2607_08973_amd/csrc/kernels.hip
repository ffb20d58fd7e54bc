// gfx950 (MI355X) kernels of the emulated SiFAR one-shot all-reduce.
//
// Work decomposition: a "chunk" is 512 consecutive bf16 elements of one
// token's row, handled by one 64-lane wave with one 16-byte load per rank per
// lane. Every chunk carries its own N epoch stamps (the paper's per-threadblock
// validation buffer, Sec. 4.2), so chunks validate and retry independently and
// no wave waits for another during the reduction proper.
//
// Two ways to run a decode step:
//  - per-epoch phases: the producer of an epoch always finishes before the
//    reduction of that epoch starts, so the paper's speculative reduction
//    (SPEC) is exact here. Eager calls and step graphs put a launch boundary
//    between the two, step_kernel (a whole step in one launch) a workgroup
//    barrier;
//  - one persistent launch per step (chain_kernel): consumer and producer
//    waves run concurrently and synchronise through stamps and per-chunk
//    consumed/produced words; the consumer validates before it loads
//    (ORDERED), since speculative loads racing a live producer were measured
//    to accept stale data.
//
// Memory-model choices (LLVM AMDGPU memory model for GFX942/950; the 8 XCDs
// have separate L2s, so agent scope means "coherent across XCDs"; the handoff
// primitives live in coherence.h, which the handoff litmus also runs):
//  - stamps are read with agent-scope atomic loads;
//  - per-epoch SPEC issues the payload loads and the stamp loads together (the
//    paper's concurrent payload warps and validation warp); ORDERED acquires
//    the stamps before loading the payload; a retry starts with an acquire
//    fence so the reloads cannot be served from a stale cache line (the
//    paper's L1-bypassing re-read, Sec. 4.2);
//  - in the persistent chain each wave learns whether its partner shares its
//    XCD. Same-XCD pairs meet in that XCD's L2: plain flag stores, a wait for
//    the slot stores instead of a release fence, agent-scope (L1-bypassing)
//    loads. Cross-XCD pairs use agent-scope stores, a release fence before the
//    stamps and an acquire fence before the payload loads.
//
// Arithmetic: fp32 adds in ascending rank order (no reassociation, no FMA
// contraction), bf16 rounding by the native V_CVT_PK_BF16_F32 (round to nearest
// even, fp32 denormals enabled).
#include "coherence.h"
#include "sifar_kernels.h"

#include <type_traits>

namespace sifar {
namespace {

__device__ __forceinline__ float lo_f32(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f32(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Two fp32 values to two bf16 in one V_CVT_PK_BF16_F32 (round to nearest
// even); converting them one at a time costs four instructions per pair.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

__device__ __forceinline__ uint32_t epoch_of(const EpochRef &e) { return e.base[0] + e.off; }

// First error wins; kind 0 means "no error".
__device__ void latch(uint32_t *err, uint32_t kind, uint32_t g, uint32_t c, uint32_t n) {
    uint32_t expected = 0;
    if (__hip_atomic_compare_exchange_strong(err, &expected, kind, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        st_relaxed(err + 1, g);
        st_relaxed(err + 2, c);
        st_relaxed(err + 3, n);
    }
}

constexpr uint32_t kErrRetryBudget = 1, kErrWaw = 2, kErrExchange = 3;

// A persistent step's waits read the error word only once they have lasted
// this many polls, and no wave reads it otherwise: a healthy epoch needs one
// or two polls, so the word is never read, while a wave whose wait outlasts
// the step's failure elsewhere still leaves within microseconds. The word is
// one address for the whole GPU: read by every consumer wave once per epoch
// (beside its first stamp poll) it bounded the step as the chunks grew.
// Measured on MI355X (llama8b decode, N = 8, H = 4096, us per all-reduce):
// reading it with every poll, 0.794 at T = 1..8 / 1.01 at 16 tokens / 2.15 at
// 64 tokens; only after 64 polls, 0.784 / 0.98 / 2.13 while consumers still
// read it once per epoch; not per epoch either, 0.760 / 0.80 / 1.12.
constexpr uint32_t kErrPollAfter = 64;

// Where the calling lane works: token t, chunk s of the row, chunk index c.
// Lanes past the end of the row load a clamped, in-bounds address (the row's
// last 8 elements) and do not store (lane_ok false) -- except where a store of
// the very bytes the owning lane stores keeps a loop branch-free; waves past
// the last chunk are inactive.
struct Chunk {
    int t, s, c;
    bool active, lane_ok;
    int elem;
    uint64_t row;
};

__device__ __forceinline__ Chunk chunk_at(const Geometry &geo, int t, int s, int lane) {
    Chunk k;
    k.t = t;
    k.active = s < geo.segs;
    k.s = k.active ? s : geo.segs - 1;
    k.c = t * geo.segs + k.s;
    const int raw = s * kChunk + lane * kVec;
    k.lane_ok = k.active && raw < geo.hidden;
    const int e = k.s * kChunk + lane * kVec;
    k.elem = e < geo.hidden ? e : geo.hidden - kVec;
    k.row = static_cast<uint64_t>(t) * geo.hidden + k.elem;
    return k;
}

__device__ __forceinline__ uint32_t log_word(uint32_t attempts, uint32_t first, uint32_t last) {
    return (attempts > 0xFFFFu ? 0xFFFFu : attempts) | ((first & 0xFFu) << 16) |
           ((last & 0xFFu) << 24);
}

// The injection table's word for epoch g (late | withheld << 8), 0 without a
// table.
__device__ __forceinline__ uint32_t inject_word(const uint16_t *inject, const DivU32 &div,
                                                uint32_t g) {
    return inject ? inject[mod_u32(g - 1u, div)] : 0u;
}

// Ranks an injection word makes late (not withheld).
__device__ __forceinline__ uint32_t late_ranks(uint32_t inj) { return inj & ~(inj >> 8) & 0xFFu; }

// ---------------------------------------------------------------------------
// Producer side: the emulated peers.

// Index of chunk k's first element in a row-major [tokens][hidden] array
// (wave-uniform), and the calling lane's byte offset from it.
__device__ __forceinline__ uint64_t chunk_first(const Geometry &geo, const Chunk &k) {
    return static_cast<uint64_t>(k.t) * geo.hidden + static_cast<uint64_t>(k.s) * kChunk;
}

__device__ __forceinline__ uint32_t lane_offset(const Geometry &geo, const Chunk &k) {
    return static_cast<uint32_t>(k.row - chunk_first(geo, k)) * 2u;
}

// Every rank's part of chunk k of epoch g (the peers' partial results), read
// through buffer descriptors: the per-lane address is the loop-invariant
// offset, so no vector register of an access in flight is ever rewritten.
template <int N>
__device__ __forceinline__ void load_sources(const ProduceArgs &a, const Chunk &k, uint32_t g,
                                             V16 (&v)[N]) {
    const uint32_t e = mod_u32(g - 1u, a.entries_div);
    const uint16_t *src = a.src + e * a.entry_stride + static_cast<int64_t>(chunk_first(a.geo, k));
    const uint32_t off = lane_offset(a.geo, k);
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = ld16_buffer<0>(src + r * a.rank_stride, off);
}

// The sources in registers, written into the slots of parity p through one
// descriptor, every rank's slot at a scalar offset from rank 0's (launch_chain
// checks that the offsets fit): one scalar instruction per store instead of
// three for a descriptor of its own, so the stores the publication waits for
// leave back to back.
template <int N>
__device__ __forceinline__ void store_slots_at(const ProduceArgs &a, const Chunk &k, uint32_t p,
                                               const V16 (&v)[N]) {
    const Geometry &geo = a.geo;
    const __amdgpu_buffer_rsrc_t rs =
        buffer_rsrc(a.slots + static_cast<uint64_t>(p) * geo.slot_elems + chunk_first(geo, k));
    const uint32_t off = lane_offset(geo, k);
    const uint32_t rank_bytes = static_cast<uint32_t>(geo.slot_elems) * 4u;
    if (k.lane_ok) {
#pragma unroll
        for (int r = 0; r < N; ++r) st16_at(rs, off, static_cast<uint32_t>(r) * rank_bytes, v[r]);
    }
}

// Copy every rank's part of chunk k of epoch g into the slots of parity p
// (the producers that load and store in one go; plain global addressing
// measured faster for them than the buffer form above). Ranks in `staged`
// (wave-uniform) write into the stage instead: they are late, and their slot
// keeps its previous epoch until they catch up.
template <int N>
__device__ __forceinline__ void copy_chunk(const ProduceArgs &a, const Chunk &k, uint32_t g,
                                           uint32_t p, uint32_t staged = 0) {
    const Geometry &geo = a.geo;
    const uint32_t e = mod_u32(g - 1u, a.entries_div);
    const uint16_t *src = a.src + e * a.entry_stride + static_cast<int64_t>(k.row);
    const uint64_t at = static_cast<uint64_t>(p) * geo.slot_elems + k.row;
    V16 v[N];
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = ld16(src + r * a.rank_stride);
    if (k.lane_ok) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            uint16_t *dst = ((staged >> r) & 1u) ? a.stage : a.slots;
            st16(dst + at + r * 2 * geo.slot_elems, v[r]);
        }
    }
}

// Ranks whose stamp an injection word holds back (late | withheld).
__device__ __forceinline__ uint32_t held_back(uint32_t inj) { return (inj | (inj >> 8)) & 0xFFu; }

// Producer of one epoch in its own launch (eager calls, step graphs). With
// deterministic injection a late rank's payload goes to the stage and its
// stamp is not written: the rank has not caught up yet. The
// stamp stores are ordered after the payload stores of the wave
// (workgroup-scope release); device-wide visibility comes from the end of the
// launch, because the reduction of an epoch always runs in a later launch than
// its producer (eagerly, in a step graph, and in the fused plane, which writes
// the epoch after the one its launch reduces) -- as in the paper, whose flag
// follows the preceding kernel's completion (Sec. 4.2). An agent-scope release
// here would write back the XCD's whole L2 once per wave; measured on MI355X
// that costs ~0.1-0.2 us of XCD-serialised time per fence and caps a 38 MB
// all-reduce at 0.9 TB/s instead of 5.7 TB/s. Workgroups are numbered
// chunk-fastest then token, the order the reduction numbers its chunks, so with
// one wave per group the producer and the reduction of a chunk share an XCD.
template <int N>
__device__ __forceinline__ void produce_chunk(const ProduceArgs &a, int G) {
    const int lane = threadIdx.x & (kLanes - 1);
    const Geometry &geo = a.geo;
    // The epoch first: the source address depends on it, and a uniform load
    // ahead of anything that may write memory stays a scalar load.
    const uint32_t g = epoch_of(a.ep);
    // Every other argument the wave reads before its source loads, requested
    // in one batch: the compiler otherwise loads kernel arguments block by
    // block, one memory round trip at a time (measured: 4-5 of them in a row
    // before the sources were requested).
    asm volatile("" ::"s"(geo.hidden), "s"(geo.segs), "s"(geo.w_max), "s"(geo.slot_elems),
                 "s"(a.ep.base), "s"(a.ep.parity), "s"(a.slots), "s"(a.stamps),
                 "s"(a.consumed), "s"(a.produced), "s"(a.src), "s"(a.entry_stride),
                 "s"(a.rank_stride), "s"(a.entries_div.m), "s"(a.entries_div.sh1),
                 "s"(a.entries_div.sh2), "s"(a.entries_div.d), "s"(a.inject), "s"(a.stage),
                 "s"(a.ep.off));
    const Chunk k = chunk_at(geo, blockIdx.y, blockIdx.x * G + threadIdx.x / kLanes, lane);
    if (!k.active) return;
    const uint32_t p = a.ep.parity;
    const size_t pc = static_cast<size_t>(p) * geo.w_max + k.c;
    // Dual-buffer rule: the slot's previous epoch must have been consumed.
    const uint32_t prev = ld_relaxed(a.produced + pc);
    const uint32_t done = ld_relaxed(a.consumed + pc);
    const uint32_t inj = inject_word(a.inject, a.inject_div, g);
    const uint32_t held = held_back(inj);
    copy_chunk<N>(a, k, g, p, a.stage ? late_ranks(inj) : 0u);
    if (lane == 0 && prev != done) latch(a.err, kErrWaw, g, k.c, prev);
    // The stamps follow the payload within the wave; the reduction reads them
    // in a later launch, whose start makes them visible device-wide, so they
    // need not be written past the L2 (an agent-scope store would make the
    // launch wait for that before it can end).
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    uint32_t *stamp = a.stamps + pc * N;
    if (lane < N && !((held >> lane) & 1u)) st_flag(stamp + lane, g, true);
    if (lane == 0) st_flag(a.produced + pc, g, true);
}

template <int N>
__global__ __launch_bounds__(1024) void produce_kernel(ProduceArgs a) {
    produce_chunk<N>(a, static_cast<int>(blockDim.x) / kLanes);
}

// ---------------------------------------------------------------------------
// Consumer side.

template <int N>
__device__ __forceinline__ void load_payload(V16 (&v)[N], const uint16_t *slot0, uint64_t rank_step) {
#pragma unroll
    for (int r = 0; r < N; ++r) v[r] = ld16(slot0 + r * rank_step);
}

// Gather of a per-epoch launch: load chunk k of epoch g, validate its N
// stamps, retry while any is stale. The epoch's on-time payload was written by
// an earlier launch, so a stale stamp can only be an injected late one.
// INJECT_HOOK: deterministic injection, the late ranks catch up right after
// the first failed validation: their payload moves from the stage into the
// slot (which still held their previous epoch when it was first loaded),
// then, after a release, their stamps are written. The retry must therefore
// reload the payload to get the right sum. `st_first` / `st_last`: this
// lane's stamp (lanes < N) at the first and at the last validation.
// `base_v` is the launch's epoch base as loaded (g = base_v + the launch's
// offset); its first use waits until the payload and stamp loads are issued.
template <int N, int MODE, bool INJECT_HOOK>
__device__ __forceinline__ uint32_t gather(const ReduceArgs &a, const Chunk &k, uint32_t base_v,
                                           uint32_t p, int lane, V16 (&v)[N], uint32_t &attempts,
                                           uint32_t &first, uint32_t &last, uint32_t &st_first,
                                           uint32_t &st_last) {
    const Geometry &geo = a.geo;
    const uint16_t *slot0 = a.slots + static_cast<uint64_t>(p) * geo.slot_elems + k.row;
    const uint64_t rank_step = 2 * geo.slot_elems;  // slots are [rank][parity]
    uint32_t *stamp = a.stamps + (static_cast<size_t>(p) * geo.w_max + k.c) * N;
    // every lane loads a stamp (lanes >= N rank N - 1's, which the ballot
    // ignores): no branch holds the loads back behind the epoch's arrival
    const uint32_t *stamp_lane = stamp + (lane < N ? lane : N - 1);

    uint32_t st = 0;
    if (MODE == kOrdered) {
        st = ld_acquire(stamp_lane);
    } else {
        load_payload<N>(v, slot0, rank_step);
        if (MODE == kSpec) st = ld_relaxed(stamp_lane);
    }
    // nothing that needs the epoch may move ahead of these loads (the compiler
    // otherwise waits for the epoch's load before it issues them)
    __builtin_amdgcn_sched_barrier(0);
    // the arguments needed once the payload is in, requested in one batch
    // while it travels (the compiler would otherwise load them one round trip
    // at a time where each is first used)
    asm volatile("" ::"s"(a.consumed), "s"(a.log), "s"(a.stamp_log), "s"(a.log_div.m),
                 "s"(a.log_div.sh1), "s"(a.log_div.sh2), "s"(a.log_div.d),
                 "s"(a.forced_retries), "s"(a.out), "s"(a.max_attempts), "s"(a.inject));
    const uint32_t g = base_v + a.ep.off;
    st_first = st;

    attempts = 1;
    first = last = 0;
    if (MODE != kNone && k.active) {
        uint32_t m = static_cast<uint32_t>(__ballot(lane < N && st != g));
        first = last = m;
        bool fail = m != 0 || a.forced_retries >= 1;
        while (fail) {
            if (attempts >= a.max_attempts) {
                if (lane == 0) latch(a.err, kErrRetryBudget, g, k.c, attempts);
                break;
            }
            if (INJECT_HOOK && attempts == 1 && a.inject && m != 0) {
                const uint32_t late = late_ranks(inject_word(a.inject, a.inject_div, g));
                if (a.stage) {
                    const uint64_t at = static_cast<uint64_t>(p) * geo.slot_elems + k.row;
#pragma unroll
                    for (int r = 0; r < N; ++r) {
                        if ((late >> r) & 1u) {
                            const V16 x = ld16(a.stage + at + r * rank_step);
                            if (k.lane_ok) st16(a.slots + at + r * rank_step, x);
                        }
                    }
                }
                // the payload is published before the stamps, as a peer would
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                if (lane < N && ((late >> lane) & 1u)) st_relaxed(stamp + lane, g);
            }
            // plain reloads need an acquire fence (an L2 invalidate) to see the
            // peers' data
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (MODE == kOrdered) {
                st = ld_acquire(stamp_lane);
            } else {
                st = ld_relaxed(stamp_lane);
                load_payload<N>(v, slot0, rank_step);
            }
            ++attempts;
            m = static_cast<uint32_t>(__ballot(lane < N && st != g));
            last = m;
            fail = m != 0 || attempts <= a.forced_retries;
        }
    }
    st_last = st;
    if (MODE == kOrdered) load_payload<N>(v, slot0, rank_step);
    return g;
}

// Persistent-step gather of an active chunk: a producer may be writing right
// now, so only ORDERED is sound. `m` is the stale-rank mask of the first stamp
// poll and `st` this lane's stamp from it (issued and evaluated by the
// caller); polls repeat (relaxed agent-scope loads; lanes >= N read rank
// N - 1's, which the ballot ignores) until every stamp is fresh, then the
// payload is loaded -- after an acquire fence when the producer is on another
// XCD, directly when it shares this XCD (see publish_slot). On return `st`
// holds the stamp of the last poll; the result is true when the wait failed:
// the retry budget ran out (latched here), or an error latched elsewhere was
// found while waiting. With AT the payload loads share one descriptor, every
// rank at a scalar offset, and leave back to back (a lone wave pays an issue
// slot for every instruction: three scalar ones per descriptor kept the last
// load ~50 ns behind the first). Measured with the producer's stores done the
// same way (llama8b decode, us per all-reduce): 0.759 -> 0.721 at T = 1..8,
// 0.80 -> 0.75 at 16 tokens, 1.13 -> 1.08 at 64 tokens. With the epilogue, whose
// scalar registers are full, it is the faster one from five ranks (8 x 8192,
// descriptor per load -> one: N = 5 1.020 -> 1.012, N = 6 1.060 -> 1.038, N = 8
// 1.083 -> 1.068; N = 8, 64 x 8192, 2.73 -> 2.70; N = 8, 128 x 8192, 7.02 -> 6.96)
// and mostly the slower one below (N = 4 0.953 -> 0.971, N = 2 0.908 -> 0.921,
// N = 3 0.964 -> 0.954), so that is the line.
template <int N, bool AT>
__device__ __forceinline__ bool gather_chain(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                             uint32_t p, int lane, uint32_t m, uint32_t &st,
                                             V16 (&v)[N], uint32_t &attempts, uint32_t &first,
                                             uint32_t &last, bool local) {
    const Geometry &geo = a.geo;
    // the chunk's first element in rank 0's slot (wave-uniform) and this
    // lane's byte offset from it
    const uint16_t *chunk0 =
        a.slots + static_cast<uint64_t>(p) * geo.slot_elems + chunk_first(geo, k);
    const uint32_t off = lane_offset(geo, k);
    const uint64_t rank_step = 2 * geo.slot_elems;  // slots are [rank][parity]
    const uint32_t *stamp = a.stamps + (static_cast<size_t>(p) * geo.w_max + k.c) * N +
                            (lane < N ? lane : N - 1);
    attempts = 1;
    first = last = m;
    bool fail = m != 0 || a.forced_retries >= 1;
    bool failed = false;
    while (fail) {
        if (attempts >= a.max_attempts) {
            if (lane == 0) latch(a.err, kErrRetryBudget, g, k.c, attempts);
            failed = true;
            break;
        }
        // one round trip per poll, back to back (a short sleep between polls
        // measured ~2 % slower); the error word joins it after kErrPollAfter
        const uint32_t e = attempts >= kErrPollAfter ? ld_relaxed(a.err) : 0u;
        st = ld_relaxed(stamp);
        ++attempts;
        m = static_cast<uint32_t>(__ballot(lane < N && st != g));
        last = m;
        if (m != 0 && e != 0) {  // the step is already failing: stop waiting
            failed = true;
            break;
        }
        fail = m != 0 || attempts <= a.forced_retries;
    }
    acquire_slot(local);
    if (AT) {
        const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(chunk0);
        const uint32_t rank_bytes = static_cast<uint32_t>(rank_step) * 2u;
#pragma unroll
        for (int r = 0; r < N; ++r)
            v[r] = ld16_agent_at(rs, off, static_cast<uint32_t>(r) * rank_bytes);
    } else {
#pragma unroll
        for (int r = 0; r < N; ++r) v[r] = ld16_agent(chunk0 + r * rank_step, off);
    }
    return failed;
}

// Fixed-order fp32 sum: acc = x_0; acc += x_1; ... acc += x_{N-1}; then bf16.
template <int N, int W>
__device__ __forceinline__ Words<W> sum_round(const Words<W> (&v)[N]) {
    float acc[2 * W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        acc[2 * k] = lo_f32(v[0].w[k]);
        acc[2 * k + 1] = hi_f32(v[0].w[k]);
    }
#pragma unroll
    for (int r = 1; r < N; ++r) {
#pragma unroll
        for (int k = 0; k < W; ++k) {
            acc[2 * k] = acc[2 * k] + lo_f32(v[r].w[k]);
            acc[2 * k + 1] = acc[2 * k + 1] + hi_f32(v[r].w[k]);
        }
    }
    Words<W> o;
#pragma unroll
    for (int k = 0; k < W; ++k) o.w[k] = pack_bf16(acc[2 * k], acc[2 * k + 1]);
    return o;
}

__device__ __forceinline__ void write_log(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                          uint32_t word) {
    a.log[static_cast<size_t>(mod_u32(g - 1u, a.log_div)) * a.geo.w_max + k.c] =
        word;
}

// Rank r's raw stamp at the chunk's first and last validation, beside the
// decision word, so that every logged mask can be recomputed from the stamps.
template <int N>
__device__ __forceinline__ void write_stamp_log(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                                int r, uint32_t first, uint32_t last) {
    uint32_t *row = a.stamp_log +
                    (static_cast<size_t>(mod_u32(g - 1u, a.log_div)) *
                         a.geo.w_max + k.c) * (2 * N) + r;
    row[0] = first;
    row[N] = last;
}

// Sum over the wave, the bit-identical total in every lane: the butterfly over
// lane distances 32, 16, 8, 4, 2, 1. The first two steps exchange half-waves
// and rows with gfx950's lane swaps; within a row of 16 a rotation by 8, 4, 2
// or 1 reaches a lane that holds the same value as the butterfly's partner
// (lanes that differ only in the bits already summed hold equal values). All
// of it stays in vector registers. A persistent epilogue step (N = 8, 8 x 8192,
// 20 all-reduces) ran at 2.33 us per all-reduce with LDS-crossbar shuffles
// here and in lanes_sum and the residual re-read every epoch; 1.67 with this
// and lane reads in lanes_sum, 1.34 with both as they are.
__device__ __forceinline__ float wave_sum(float v) {
    auto pair = [](auto r) { return __uint_as_float(r[0]) + __uint_as_float(r[1]); };
    const auto bits = [](float x) { return __float_as_uint(x); };
    v = pair(__builtin_amdgcn_permlane32_swap(bits(v), bits(v), false, false));
    v = pair(__builtin_amdgcn_permlane16_swap(bits(v), bits(v), false, false));
    auto ror = [&](auto ctrl) {
        const int x = static_cast<int>(bits(v));
        v = v + __uint_as_float(static_cast<uint32_t>(
                    __builtin_amdgcn_update_dpp(x, x, decltype(ctrl)::value, 0xF, 0xF, true)));
    };
    ror(std::integral_constant<int, 0x128>{});  // row_ror:8
    ror(std::integral_constant<int, 0x124>{});
    ror(std::integral_constant<int, 0x122>{});
    ror(std::integral_constant<int, 0x121>{});
    return v;
}

// Sum of lanes 0 .. n - 1 of v (the token's n exchange words), in every lane. The
// butterfly again: adding the 16 words of an 8192-wide token in lane order
// took 16 LDS-crossbar shuffles, or 16 dependent lane reads (below).
__device__ __forceinline__ float lanes_sum(float v, int n, int lane) {
    return wave_sum(lane < n ? v : 0.f);
}

// Residual-add + RMSNorm of one chunk after its all-reduce result o. The
// token's sum of squares is combined across the waves of the workgroup (LDS)
// and across the token's Q workgroups (epoch-tagged exchange words, double
// buffered by the epoch's parity). Every wave of the workgroup must call this.
__device__ __forceinline__ void residual_rmsnorm(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                                 const V16 &o, const V16 &rv,
                                                 const V16 &wv, uint16_t *y, int lane, int wave,
                                                 int G, int q) {
    const Geometry &geo = a.geo;
    // res' = bf16(a + res), with a = the bf16 all-reduce result.
    V16 nr;
    float x[kVec];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a0 = lo_f32(o.w[i]), a1 = hi_f32(o.w[i]);
        nr.w[i] = pack_bf16(a0 + lo_f32(rv.w[i]), a1 + hi_f32(rv.w[i]));
        x[2 * i] = lo_f32(nr.w[i]);
        x[2 * i + 1] = hi_f32(nr.w[i]);
    }
    if (k.lane_ok) st16(a.residual + k.row, nr);

    float ss = 0.f;
    if (k.lane_ok) {
#pragma unroll
        for (int i = 0; i < kVec; ++i) ss = __builtin_fmaf(x[i], x[i], ss);
    }
    ss = wave_sum(ss);

    __shared__ float part[kMaxWavesPerGroup];
    __shared__ float total;
    if (lane == 0) part[wave] = ss;  // idle waves contribute 0
    __syncthreads();
    float grp = 0.f;
    for (int w = 0; w < G; ++w) grp = grp + part[w];

    const int Q = a.groups_per_token;
    if (Q > 1) {
        if (wave == 0) {
            uint64_t *ex = a.exch + static_cast<size_t>(g & 1u) * a.exch_parity_stride +
                           static_cast<size_t>(k.t) * Q;
            if (lane == 0) {
                const uint64_t word = (static_cast<uint64_t>(g) << 32) | __float_as_uint(grp);
                __hip_atomic_store(ex + q, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            uint64_t mine = 0;
            uint32_t spins = 0;
            bool ready;
            do {
                if (lane < Q)
                    mine = __hip_atomic_load(ex + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ready = __ballot(lane < Q && static_cast<uint32_t>(mine >> 32) != g) == 0;
            } while (!ready && ++spins < a.spin_limit);
            if (!ready && lane == 0) latch(a.err, kErrExchange, g, k.c, spins);
            const float tot = lanes_sum(__uint_as_float(static_cast<uint32_t>(mine)), Q, lane);
            if (lane == 0) total = tot;
        }
        __syncthreads();
        grp = total;
    }

    const float inv = 1.0f / __builtin_sqrtf(grp / static_cast<float>(geo.hidden) + a.eps);
    V16 yo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float w0 = lo_f32(wv.w[i]), w1 = hi_f32(wv.w[i]);
        yo.w[i] = pack_bf16((x[2 * i] * inv) * w0, (x[2 * i + 1] * inv) * w1);
    }
    if (k.lane_ok) st16(y + k.row, yo);
}

// ---------------------------------------------------------------------------
// Reduction of one epoch, one chunk per wave: speculative or ordered loads,
// per-rank stamp validation by ballot, bounded retry, fp32 sum in rank order,
// bf16 store, optional fused epilogue.
// FUSED: the grid has a second plane (blockIdx.z == 1) of producer workgroups
// that write the NEXT epoch (other parity) while the first plane reduces this
// one -- the emulated peers running one epoch ahead, which is as far ahead as
// two slots allow. The planes touch disjoint slots and stamps.
//
// The arguments both planes need first come as the kernel's leading scalar
// arguments: gfx950 can preload leading kernel arguments into scalar
// registers when a wave starts (the build asks the compiler for it), so the
// epoch's location and the slot and stamp addresses are known without a
// memory round trip. `shape` packs hidden (bits 0-16), chunks per token (bits
// 17-24), the consumer's slot parity (bit 25) and log2 of the waves per
// workgroup (bits 26-28). The structs carry the rest, read later.
template <int N, int MODE, bool EPI, bool FUSED>
__global__ __launch_bounds__(1024) void reduce_kernel(const uint32_t *ep_base, uint16_t *slots,
                                                      uint32_t *stamps, uint64_t slot_elems,
                                                      uint32_t shape, uint32_t w_max,
                                                      uint32_t ep_off, ReduceArgs ra,
                                                      ProduceArgs pa) {
    const int hidden = static_cast<int>(shape & 0x1FFFFu);
    const int segs = static_cast<int>((shape >> 17) & 0xFFu);
    const int G = 1 << ((shape >> 26) & 7u);
    if (FUSED && blockIdx.z == 1) {
        ProduceArgs pp = pa;
        pp.geo.hidden = hidden;
        pp.geo.segs = segs;
        pp.geo.w_max = static_cast<int32_t>(w_max);
        pp.geo.slot_elems = slot_elems;
        pp.ep.base = ep_base;
        pp.slots = slots;
        pp.stamps = stamps;
        produce_chunk<N>(pp, G);
        return;
    }
    ReduceArgs a = ra;
    a.geo.hidden = hidden;
    a.geo.segs = segs;
    a.geo.w_max = static_cast<int32_t>(w_max);
    a.geo.slot_elems = slot_elems;
    a.ep.base = ep_base;
    a.ep.off = ep_off;
    a.ep.parity = (shape >> 25) & 1u;
    a.slots = slots;
    a.stamps = stamps;
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = threadIdx.x / kLanes;
    const Geometry &geo = a.geo;
    // The epoch base is read first: its address is at hand, and a uniform
    // load ahead of anything that may write memory stays a scalar load.
    const uint32_t base_v = ep_base[0];
    // grid: x = chunk groups of a token, y = token
    const Chunk k = chunk_at(geo, blockIdx.y, blockIdx.x * G + wave, lane);
    if (!EPI && !k.active) return;  // EPI: idle waves still join the barriers
    const uint32_t p = a.ep.parity;

    V16 rv, wv;
    if (EPI) {
        rv = ld16(a.residual + k.row);
        wv = ld16(a.weight + k.elem);
    }
    V16 v[N];
    uint32_t attempts, first, last, st_first, st_last;
    const uint32_t g =
        gather<N, MODE, true>(a, k, base_v, p, lane, v, attempts, first, last, st_first, st_last);
    const V16 o = sum_round<N, 4>(v);
    if (k.active && lane == 0) {
        write_log(a, k, g, log_word(attempts, first, last));
        a.consumed[static_cast<size_t>(p) * geo.w_max + k.c] = g;
    }
    if (a.stamp_log && k.active && lane < N) write_stamp_log<N>(a, k, g, lane, st_first, st_last);
    if (!EPI) {
        if (k.lane_ok) st16_stream(a.out + k.row, o);
        return;
    }
    residual_rmsnorm(a, k, g, o, rv, wv, a.y, lane, wave, G, blockIdx.x);
}

// The epilogue of a step in one launch in two halves, so that the wait for the
// token's other waves overlaps the next epoch's reduction instead of
// stalling every chunk of the token once per epoch. Only the residual carries
// from one epoch to the next, and it is this chunk's own (it stays in
// registers for the whole step and is stored at its end); the token-wide sum
// of squares is needed for y alone. epi_stage runs right after epoch g's sum:
// it updates the residual, reduces this wave's sum of squares and publishes
// it in exchange plane g mod kExchPlanes. epi_finish runs one epoch later, or
// after the step's last epoch: it takes the token's Q words of epoch g,
// adds them (lanes_sum) and writes y. The arithmetic is residual_rmsnorm's.
// Four planes suffice: a wave can publish epoch g + 4 only after finishing
// epoch g + 2, which needs every wave's word of g + 2, and a wave publishes
// that only after it finished epoch g.
template <int W>
struct EpiPending {
    Words<W> res;  // res' of this lane's elements
    float sum;     // this wave's sum of squares
    uint32_t g;    // the epoch
};

template <int W>
__device__ __forceinline__ void epi_stage(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                          const Words<W> &o, Words<W> &res, int lane, int q,
                                          bool xlocal, EpiPending<W> &pd) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const float a0 = lo_f32(o.w[i]), a1 = hi_f32(o.w[i]);
        res.w[i] = pack_bf16(a0 + lo_f32(res.w[i]), a1 + hi_f32(res.w[i]));
        const float x0 = lo_f32(res.w[i]), x1 = hi_f32(res.w[i]);
        ss = __builtin_fmaf(x0, x0, ss);
        ss = __builtin_fmaf(x1, x1, ss);
    }
    ss = wave_sum(k.lane_ok ? ss : 0.f);
    pd.res = res;

    pd.sum = ss;
    pd.g = g;

    const int Q = a.groups_per_token;
    if (Q > 1 && lane == 0) {
        uint64_t *ex = a.exch + static_cast<size_t>(g % kExchPlanes) * a.exch_parity_stride +
                       static_cast<size_t>(k.t) * Q;
        const uint64_t word = (static_cast<uint64_t>(g) << 32) | __float_as_uint(ss);
        // all waves of the token on this XCD: the word meets them in its L2
        if (xlocal)
            __hip_atomic_store(ex + q, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_store(ex + q, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// This lane's exchange word of epoch g (lanes >= Q read wave Q - 1's).
__device__ __forceinline__ uint64_t epi_word(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                             int lane) {
    const int Q = a.groups_per_token;
    const uint64_t *ex = a.exch + static_cast<size_t>(g % kExchPlanes) * a.exch_parity_stride +
                         static_cast<size_t>(k.t) * Q;
    return __hip_atomic_load(ex + (lane < Q ? lane : Q - 1), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
}

// `y` is the ring entry of epoch pd.g, `mine` this lane's exchange word of it
// as loaded before the reduction of the epoch after (usually every wave's is
// there by then). (`pd` by value: with a reference the
// compiler kept the pending state in scratch memory.) True when the
// exchange wait failed: it ran out of polls (latched here), or found an error
// latched elsewhere.
template <int W>
__device__ __forceinline__ bool epi_finish(const ReduceArgs &a, const Chunk &k,
                                           const EpiPending<W> pd, uint64_t mine,
                                           const Words<W> &wv, uint16_t *y, int lane) {
    const int Q = a.groups_per_token;
    float tot = pd.sum;
    bool failed = false;
    if (Q > 1) {
        uint32_t spins = 0;
        bool ready = __ballot(static_cast<uint32_t>(mine >> 32) != pd.g) == 0;
        while (!ready) {
            if (spins >= kErrPollAfter && ld_relaxed(a.err) != 0) break;
            if (++spins >= a.spin_limit) break;
            mine = epi_word(a, k, pd.g, lane);
            ready = __ballot(static_cast<uint32_t>(mine >> 32) != pd.g) == 0;
        }
        failed = !ready;
        if (!ready && lane == 0) latch(a.err, kErrExchange, pd.g, k.c, spins);
        tot = lanes_sum(__uint_as_float(static_cast<uint32_t>(mine)), Q, lane);
    }
    const float inv = 1.0f / __builtin_sqrtf(tot / static_cast<float>(a.geo.hidden) + a.eps);
    Words<W> yo;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const float w0 = lo_f32(wv.w[i]), w1 = hi_f32(wv.w[i]);
        yo.w[i] = pack_bf16((lo_f32(pd.res.w[i]) * inv) * w0, (hi_f32(pd.res.w[i]) * inv) * w1);
    }
    if (k.lane_ok) st_words<W>(y + k.row, yo);
    return failed;
}

// ---------------------------------------------------------------------------
// Persistent decode step: one launch runs all L all-reduces. All waves are
// co-resident (the host checks), and every wait is bounded.
//
// Per chunk and epoch g of parity p:
//   producer  wait until consumed[p] == produced[p] (the reduction that read
//             this slot two epochs back has finished: dual buffering), copy
//             the N partials, publish them (publish_slot: a release fence
//             only when the consumer is on another XCD), store the on-time
//             stamps and produced[p] = g; injected late ranks' stamps follow
//             after `late_delay` sleeps.
//   consumer  poll the stamps (relaxed agent-scope loads, back to back) until
//             all are fresh, then load the payload (after an acquire fence
//             when the producer is on another XCD); sum; store; consumed[p] =
//             g once every payload load has completed.
// Every wait is bounded, and joins the error word to its polls only once it
// has lasted kErrPollAfter polls.
// Validation comes before the payload loads here (ORDERED). Speculative
// payload loads issued alongside the stamp loads were measured to return a
// rank's previous epoch while its stamp already read as fresh when producer
// and consumer sat on different XCDs: the monotonicity the paper assumes
// (Sec. 8.1) does not hold for a live producer on MI355X. (The per-epoch
// launches keep SPEC: there every epoch was written by an earlier launch.)
// The producer can run one epoch ahead of the consumer, no further.
// Producer wave of chunk (t, s), one epoch after the other: wait until the
// slot of this parity is free (with a single buffer: until the previous
// epoch's reduction is done -- the bottom barrier), store the sources already
// in registers, publish, stamps. Loading the next epoch's sources while the
// slot stores travel shortened the llama8b decode step by ~5 % on MI355X once
// the consumer issued its polls ahead of its stores; before that the consumer
// bounded the step and the prefetch made no difference.
template <int N, bool PREFETCH>
__device__ __forceinline__ void chain_producer(const ChainArgs &A, uint32_t base, int lane,
                                               int bx, int by) {
    const ProduceArgs &a = A.p;
    const Geometry &geo = a.geo;
    const Chunk k = chunk_at(geo, by, bx, lane);
    publish_place(A.place + geo.w_max + k.c, base, lane);
    const bool local = partner_is_local(A.place + k.c, base, lane);
    // One epoch: wait until the slot is free, store `cur` (the epoch's
    // sources, already in registers), load the next epoch's sources into
    // `nxt` while the slot stores travel (harmless in-bounds reads after the
    // last epoch), publish, stamp. False when the slot wait failed.
    auto epoch = [&](int i, const V16(&cur)[N], V16(&nxt)[N]) -> bool {
        const uint32_t g = base + static_cast<uint32_t>(i) + 1u;
        const uint32_t p = static_cast<uint32_t>(i + 1) & A.parity_mask;
        const size_t pc = static_cast<size_t>(p) * geo.w_max + k.c;
        uint32_t spins = 0;
        bool free = false;
        // one round trip per poll: both words together, and the error word
        // after kErrPollAfter polls; a short sleep between polls (without it
        // the kernel takes 109 VGPRs instead of 76 and the step ran ~0.6 %
        // slower)
        while (true) {
            const uint32_t done = ld_relaxed(a.consumed + pc);
            const uint32_t prev = ld_relaxed(a.produced + pc);
            const uint32_t e = spins >= kErrPollAfter ? ld_relaxed(a.err) : 0u;
            free = done == prev;
            if (free || ++spins >= A.r.spin_limit || e != 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if (!free) {
            if (lane == 0) latch(a.err, kErrWaw, g, k.c, spins);
            return false;
        }
        const uint32_t inj = inject_word(a.inject, a.inject_div, g);
        const uint32_t held = held_back(inj);
        if (!PREFETCH) {
            copy_chunk<N>(a, k, g, p);
            publish_slot(local);
        } else if (local) {
            store_slots_at<N>(a, k, p, cur);
            // the loads stay after the stores (the wait below counts on it)
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            load_sources<N>(a, k, g + 1u, nxt);
            // Loads and stores complete in issue order on gfx9-family GPUs:
            // with at most N operations outstanding the slot stores have
            // reached the L2 and only the N source loads are still in flight.
            __builtin_amdgcn_s_waitcnt(kWaitVm | N);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
        } else {
            store_slots_at<N>(a, k, p, cur);
            load_sources<N>(a, k, g + 1u, nxt);
            publish_slot(false);
        }
        uint32_t *stamp = a.stamps + pc * N;
        if (lane < N && !((held >> lane) & 1u)) st_flag(stamp + lane, g, local);
        if (lane == 0) st_flag(a.produced + pc, g, local);
        if (held) {
            for (uint32_t d = 0; d < A.late_delay; ++d) __builtin_amdgcn_s_sleep(8);
            if (lane < N && ((inj >> lane) & 1u) && !((inj >> (8 + lane)) & 1u))
                st_flag(stamp + lane, g, local);
        }
        return true;
    };
    // Two register sets taking turns: a load never overwrites the data of a
    // store still in flight, so nothing waits for the store acknowledgements
    // before the next sources are requested. (Without PREFETCH every epoch
    // loads and stores in one go: 2N fewer registers, for steps whose waves
    // fit on the GPU only at the higher occupancy.)
    V16 va[N], vb[N];
    if (PREFETCH) load_sources<N>(a, k, base + 1u, va);
    for (int i = 0; i < A.reduces; i += 2) {
        if (!epoch(i, va, vb)) return;
        if (i + 1 < A.reduces && !epoch(i + 1, vb, va)) return;
    }
}

// Consumer wave of chunk (t, x).
template <int N, int MODE, bool EPI>
__device__ __forceinline__ void chain_consumer(const ChainArgs &A, uint32_t base, int lane, int bx,
                                               int by) {
    const ReduceArgs &a = A.r;
    const Geometry &geo = a.geo;
    const Chunk k = chunk_at(geo, by, bx, lane);
    // (every wave has a chunk; with the test the compiler schedules the epilogue's
    // loop 1.5 % faster)
    if (k.active) publish_place(A.place + k.c, base, lane);
    const bool local = k.active && partner_is_local(A.place + geo.w_max + k.c, base, lane);
    // the epilogue's exchange partners: the consumers of this token's chunks
    bool xlocal = false;
    if (EPI) {
        const int Q = a.groups_per_token;
        const bool mine = lane >= Q ||
                          tag_is_local(A.place + static_cast<size_t>(k.t) * geo.segs + lane, base);
        xlocal = __ballot(!mine) == 0;
    }
    V16 wv, res;
    if (EPI) {
        wv = ld16(a.weight + k.elem);
        res = ld16(a.residual + k.row);
    }
    EpiPending<4> pending;  // the epilogue of the previous epoch, finished one epoch late
    bool have_pending = false;
    // Every lane polls a stamp of this chunk (lanes >= N repeat rank N - 1's,
    // which the ballot ignores), so no branch surrounds the poll.
    const uint32_t *stamps = a.stamps + static_cast<size_t>(k.c) * N + (lane < N ? lane : N - 1);
    const size_t parity_stride = static_cast<size_t>(geo.w_max) * N;
    // The first poll of an epoch -- its stamps -- is issued before the
    // previous epoch's stores. On gfx9-family GPUs one counter
    // (vmcnt) tracks loads and stores in issue order, so a poll issued after
    // the stores could only be waited for together with their write
    // acknowledgements. The stores below are therefore branch-free too, so the
    // compiler can count them and wait for the poll alone. An early poll that
    // reads stale is repeated; the payload is still loaded only after fresh
    // stamps were seen.
    uint32_t st_next = ld_relaxed(stamps + (1u & A.parity_mask) * parity_stride);
    // stale ranks of the first poll, evaluated where the wait for it is exact
    uint32_t m_next = static_cast<uint32_t>(__ballot(lane < N && st_next != base + 1u));
    for (int i = 0; i < A.reduces; ++i) {
        const uint32_t g = base + static_cast<uint32_t>(i) + 1u;
        const uint32_t p = static_cast<uint32_t>(i + 1) & A.parity_mask;
        uint64_t word = 0;  // the pending epoch's exchange word
        if (EPI && have_pending) word = epi_word(a, k, pending.g, lane);
        V16 v[N];
        uint32_t attempts, first, last;
        const uint32_t st_first = st_next;
        uint32_t st_last = st_next;
        bool stop =
            gather_chain<N, !EPI || (N > 4)>(a, k, g, p, lane, m_next, st_last, v, attempts, first, last, local);
        uint32_t *consumed = a.consumed + static_cast<size_t>(p) * geo.w_max + k.c;
        // Once the payload has arrived: issue the next epoch's first poll (a
        // harmless in-bounds read after the last epoch), then release the slot
        // (every lane stores the same word).
        auto poll_next_and_release = [&]() {
            const uint32_t pn = static_cast<uint32_t>(i + 2) & A.parity_mask;
            st_next = ld_relaxed(stamps + pn * parity_stride);
            __atomic_signal_fence(__ATOMIC_SEQ_CST);  // keep the poll ahead of the stores
            st_flag(consumed, g, local);
        };
        if (!EPI) {
            // release the slot as soon as every payload load has returned (the
            // sum works on registers); with the epilogue that is the slower one
            // (N = 8, 8 x 8192: 1.18 us per all-reduce, after the sum 1.10; N =
            // 2, 64 x 8192: 1.13 and 1.12)
#pragma unroll
            for (int r = 0; r < N; ++r) complete(v[r]);
            poll_next_and_release();
        }
        const V16 o = sum_round<N, 4>(v);
        if (EPI) {
            complete(o);  // every payload load has returned before the slot is released
            poll_next_and_release();
        }
        write_log(a, k, g, log_word(attempts, first, last));  // wave-uniform word
        // lanes >= N store rank N - 1's stamps again: the same words to the same place
        write_stamp_log<N>(a, k, g, lane < N ? lane : N - 1, st_first, st_last);
        const uint64_t ring = static_cast<uint64_t>(i) * A.ring_stride;
        if (!EPI) {
            // Lanes past the end of the row loaded the row's last 8 elements
            // (clamped) with the same instruction as the lane that owns them,
            // so they store the same bytes to the same place: no branch.
            st16_stream(a.out + ring + k.row, o);
        } else {
            EpiPending<4> cur;
            epi_stage<4>(a, k, g, o, res, lane, bx, xlocal, cur);
            if (have_pending &&
                epi_finish<4>(a, k, pending, word, wv, a.y + ring - A.ring_stride, lane))
                stop = true;
            pending = cur;
            have_pending = true;
        }
        // The next epoch's first poll, after this epoch's stores: the
        // compiler waits for the poll alone and leaves the stores in flight.
        m_next = static_cast<uint32_t>(__ballot(lane < N && st_next != g + 1u));
        // a bounded wait of this wave failed: stop (a pending epilogue stays
        // unwritten: the step has failed). Every wait is bounded and reads the
        // error word once it has lasted kErrPollAfter polls, so a failure
        // anywhere ends the other waves' waits too.
        if (stop) {
            if (EPI && k.lane_ok) st16(a.residual + k.row, res);
            return;
        }
    }
    if (EPI) {
        if (k.lane_ok) st16(a.residual + k.row, res);
        epi_finish<4>(a, k, pending, epi_word(a, k, pending.g, lane), wv,
                      a.y + static_cast<uint64_t>(A.reduces - 1) * A.ring_stride, lane);
    }
}

// Grid (segs, plane_rows(tokens, segs), 2) of one-wave workgroups, or with the
// epilogue (8 * ceil(tokens / 8) * segs, 1, 2), layout below: plane 0 reduces
// chunk (t, x) for epochs base+1 .. base+L in order, plane 1 produces it. The
// last wave to arrive on the counter advances the epoch base for the next
// step: every wave read the base before it arrived, so no wave can see the
// advanced value. (The occupancy asked for with the epilogue keeps the largest
// steps that init accepts where they were.)
//
// Epilogue steps from 512 chunks on once ran four-wave workgroups that shared a
// slot publication and an exchange word, with barriers between their waves.
// With the sums in vector registers and the residual kept there, one wave per
// workgroup is the faster one at every size (us per all-reduce, four waves ->
// one): N = 8, 32 x 8192, 2.12 -> 1.24; 64 x 8192, 2.92 -> 2.81; 160 x 8192,
// 8.84 both; N = 4, 32 x 8192, 1.84 -> 1.06; N = 2, 64 x 8192, 1.83 -> 1.11; one
// buffer, N = 8, 32 x 8192, 2.44 -> 1.59, 128 x 8192, 5.37 -> 5.40.
template <int N, int MODE, bool EPI, bool PREFETCH>
__global__ __launch_bounds__(kLanes, EPI ? 5 : 1) void chain_kernel(ChainArgs A) {
    const int lane = threadIdx.x & (kLanes - 1);
    const uint32_t base = A.r.ep.base[0];
    // Logical (chunk, token). With the epilogue, workgroup b of a plane serves
    // token (b mod 8) + 8 * (b / 8 / segs), chunk (b / 8) mod segs: every chunk
    // of a token -- consumers and producers, since each plane holds a multiple
    // of 8 workgroups -- is dealt to the same XCD, so the per-epoch exchange of
    // the token's sum of squares stays in one L2. Workgroups past the last
    // token only arrive on the counter.
    int bx = blockIdx.x, by = blockIdx.y;
    if (EPI) {
        const int Q = A.r.groups_per_token;
        const int j = static_cast<int>(blockIdx.x) >> 3;
        bx = j % Q;
        by = (static_cast<int>(blockIdx.x) & 7) + 8 * (j / Q);
    }
    if (by < A.r.geo.tokens) {
        if (blockIdx.z == 1)
            chain_producer<N, PREFETCH>(A, base, lane, bx, by);
        else
            chain_consumer<N, MODE, EPI>(A, base, lane, bx, by);
    }
    if (lane == 0) {
        const uint32_t waves = 2u * gridDim.x * gridDim.y;
        const uint32_t before =
            __hip_atomic_fetch_add(A.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == waves - 1u) {
            st_relaxed(A.done, 0u);
            st_relaxed(A.epoch_base, base + A.advance);
        }
    }
}

// ---------------------------------------------------------------------------
// Per-epoch step in one launch: every all-reduce of a decode step, with a
// workgroup barrier where the step graph has a launch boundary.
//
// A workgroup is one chunk: its first wave (or first four, a quarter of the
// chunk's elements each) is the consumer, its last plays the peers. Phase i:
// the peers write epoch base + i + 1 while the consumer reduces epoch base +
// i; the barrier between phases orders them as the end of a launch would, so
// speculation is as exact here as there: whatever the consumer loads in a
// phase was written before the barrier. Chunks share nothing, so no workgroup
// waits for another. Barrier and loads stay on one CU: the peers' stores need
// no acknowledgement and no release fence before the barrier, the consumer's
// loads follow them through the CU's memory pipeline and are served by the
// XCD's L2 (agent scope: past the L1).
//
// What bounds it: the consumer's phase, one L2 round trip (payload and stamps
// together), the rest of the sum that the loads' arrival does not cover, and
// the issue of its stores; from 1024 chunks at N = 8 the bytes. Measured
// against one launch per all-reduce (us per all-reduce, launches -> one
// launch, one consumer wave): N = 8, 4 tokens x 4096, 64 per step, 2.62 ->
// 0.58; with 10 % late stamps 3.70 -> 1.12; 20 per step: N = 2, 1 x 4096, 2.59
// -> 0.49; N = 8, 64 x 4096, 3.69 -> 1.14; 64 x 8192, 5.49 -> 3.04; 256 x 8192
// (4096 chunks, every wave slot of the GPU), 16.3 -> 14.0; N = 2, 256 x 8192,
// 6.46 -> 3.92. With the epilogue: 1 x 4096, 4.57 -> 1.13; 40 x 8192, 7.21 ->
// 1.71; 32 x 8192 with 5 % late stamps, 120 per step, 10.6 -> 1.68. It is the
// faster one wherever its workgroups fit at once, so that is the rule (with the
// epilogue up to a quarter of that, see sifar_init); beyond that, chunks would
// run their whole step one after another, which no sequence of all-reduces
// does.
// INJECT: the kernel that knows the injection table; without one the table's
// branches leave the scalar registers (and 5 % of the time).
//
// Four consumer waves: the sum is ~130 vector instructions of a wave, 0.2 us,
// of which the payload's arrival covers a fourth; split four ways it is nearly
// hidden. No wave waits for a partner's poll here (the barrier is there
// anyway), which is what makes the split pay. Measured, one -> four (64
// all-reduces, us per all-reduce): N = 8, 8 chunks 0.573 -> 0.517, 128 chunks
// 0.601 -> 0.533, 256 chunks 0.644 -> 0.576; N = 4, 64 chunks 0.455 -> 0.420;
// N = 2, 64 chunks 0.396 -> 0.390; with the epilogue 128 chunks 1.03 -> 0.90.
// At 512 chunks it is 0.803 -> 0.740 (N = 8, rows of 4096) but 0.99 -> 1.01
// (N = 5, ragged rows of 3896), at 1024 2.75 -> 2.74. (Two waves were slower
// than one at N = 4 and 8: 0.58 -> 0.63.) So steps split up to 256 chunks, one
// per CU; epilogue steps no further than a quarter of the places of the wider
// workgroup.

// Phase boundary: orders the workgroup's memory operations on their CU.
__device__ __forceinline__ void phase_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The peers of one chunk. `done` (LDS): the last epoch of each parity that the
// consumer of this launch has finished; the first epoch of each parity checks
// the words that earlier launches left in memory. Sources, slots and stage are
// each addressed through one descriptor, every rank at a scalar offset (the
// host checks that they fit 31 bits): pointers per rank overflow the scalar
// registers. (Only the late ranks' stage stores choose a descriptor each: two
// descriptors and a lane offset per rank, as in catch_up, were 5 % slower
// here.)
template <int N, bool INJECT, int C>
__device__ __forceinline__ void step_producer(const ChainArgs &A, uint32_t base, const Chunk &k,
                                              int lane, uint32_t (&done)[2][C]) {
    const ProduceArgs &a = A.p;
    const Geometry &geo = a.geo;
    const uint32_t off = lane_offset(geo, k);
    const uint64_t first = chunk_first(geo, k);
    const uint32_t rank_bytes = static_cast<uint32_t>(geo.slot_elems) * 4u;
    const uint32_t src_bytes = static_cast<uint32_t>(a.rank_stride) * 2u;
    V16 v[N];
    auto load = [&](uint32_t g) {
        const uint32_t e = mod_u32(g - 1u, a.entries_div);
        const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(a.src + e * a.entry_stride + first);
#pragma unroll
        for (int r = 0; r < N; ++r) v[r] = ld16_at(rs, off, static_cast<uint32_t>(r) * src_bytes);
    };
    // Dual-buffer rule: a slot's previous epoch must have been consumed. The
    // step's first two epochs follow earlier launches' words, which travel with
    // the first sources (a round trip of their own ahead of them cost 0.5 us a
    // step), as does the injection word.
    const uint32_t prev1 = ld_relaxed(a.produced + geo.w_max + k.c);
    const uint32_t fin1 = ld_relaxed(a.consumed + geo.w_max + k.c);
    const uint32_t prev2 = ld_relaxed(a.produced + k.c);
    const uint32_t fin2 = ld_relaxed(a.consumed + k.c);
    uint32_t word = 0;
    if (INJECT) word = inject_word(a.inject, a.inject_div, base + 1u);
    load(base + 1u);
    if (lane == 0) {
        if (prev1 != fin1) latch(a.err, kErrWaw, base + 1u, k.c, prev1);
        if (A.reduces > 1 && prev2 != fin2) latch(a.err, kErrWaw, base + 2u, k.c, prev2);
    }
    for (int i = 0; i < A.reduces; ++i) {
        const uint32_t g = base + static_cast<uint32_t>(i) + 1u;
        const uint32_t p = static_cast<uint32_t>(i + 1) & 1u;
        const size_t pc = static_cast<size_t>(p) * geo.w_max + k.c;
        const uint64_t at = static_cast<uint64_t>(p) * geo.slot_elems + first;
        if (i >= 2) {
            const uint32_t fin = __hip_atomic_load(&done[p][lane % C], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            if (lane < C && fin != g - 2u) latch(a.err, kErrWaw, g, k.c, g - 2u);
        }
        const uint32_t inj = INJECT ? __builtin_amdgcn_readfirstlane(word) : 0u;
        const uint32_t staged = late_ranks(inj);
        const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(a.slots + at);
        // lanes past the row's end store the owning lane's bytes again: no
        // branch, so nothing in flight is waited for beyond the data stored
        if (!INJECT || staged == 0) {
#pragma unroll
            for (int r = 0; r < N; ++r)
                st16_at(rs, off, static_cast<uint32_t>(r) * rank_bytes, v[r]);
        } else {
#pragma unroll
            for (int r = 0; r < N; ++r)
                st16_at(buffer_rsrc((((staged >> r) & 1u) ? a.stage : a.slots) + at), off,
                        static_cast<uint32_t>(r) * rank_bytes, v[r]);
        }
        // the stamps follow the payload
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane < N && !((held_back(inj) >> lane) & 1u)) st_flag(a.stamps + pc * N + lane, g, true);
        if (lane == 0) st_flag(a.produced + pc, g, true);
        // the next epoch's sources travel while the consumer works (after the
        // last epoch: harmless reads of the pool)
        if (INJECT) word = inject_word(a.inject, a.inject_div, g + 1u);
        load(g + 1u);
        phase_barrier();
    }
}

// Moves the late ranks' payload of a chunk from the stage into the slots, then
// their stamps: the ranks catch up. The stage and the slots have one descriptor
// each; a descriptor per late rank and side took 64 scalar registers at N = 8,
// and up to 55 were spilled (now 36).
template <int N>
__device__ __forceinline__ void catch_up(const ReduceArgs &a, const Chunk &k, uint32_t g,
                                         uint32_t p, uint32_t late, int lane, uint32_t *stamp) {
    const uint32_t rank_bytes = static_cast<uint32_t>(a.geo.slot_elems) * 4u;
    const uint64_t at = static_cast<uint64_t>(p) * a.geo.slot_elems + chunk_first(a.geo, k);
    const uint32_t off = lane_offset(a.geo, k);
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(a.slots + at), rt = buffer_rsrc(a.stage + at);
    V16 x[N];
#pragma unroll
    for (int r = 0; r < N; ++r)
        x[r] = ld16_at(rt, offset_if(off, (late >> r) & 1u), static_cast<uint32_t>(r) * rank_bytes);
#pragma unroll
    for (int r = 0; r < N; ++r)
        st16_at(rs, offset_if(off, (late >> r) & 1u), static_cast<uint32_t>(r) * rank_bytes, x[r]);
    // the payload is published before the stamps, as a peer would; both are
    // read again by this wave alone
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane < N && ((late >> lane) & 1u)) st_flag(stamp + lane, g, true);
}

// Where lane `lane` of consumer wave w of C works: its 8 / C elements of the
// chunk, as chunk_at places them for one wave.
template <int C>
__device__ __forceinline__ Chunk part_of(const Geometry &geo, Chunk k, int w, int lane) {
    const int raw = k.s * kChunk + w * (kChunk / C) + lane * (kVec / C);
    k.lane_ok = raw < geo.hidden;
    k.elem = k.lane_ok ? raw : geo.hidden - kVec / C;
    k.row = static_cast<uint64_t>(k.t) * geo.hidden + k.elem;
    return k;
}

// Consumer wave w of C. Each validates its part's stamps itself; wave 0 keeps the
// log (without injection no stamp is ever stale, so the waves cannot differ).
template <int N, int MODE, bool EPI, bool INJECT, int C>
__device__ __forceinline__ void step_consumer(const ChainArgs &A, uint32_t base, const Chunk &kc,
                                              int w, int lane, uint32_t (&done)[2][C]) {
    static_assert(!INJECT || C == 1, "late ranks catch up in one consumer wave");
    constexpr int W = 4 / C;
    const ReduceArgs &a = A.r;
    const Geometry &geo = a.geo;
    const Chunk k = part_of<C>(geo, kc, w, lane);
    const uint32_t off = lane_offset(geo, k);
    const uint32_t rank_bytes = static_cast<uint32_t>(geo.slot_elems) * 4u;
    // the epilogue as in the persistent step: finished one epoch late
    bool xlocal = false;
    Words<W> wv, res;
    EpiPending<W> pending;
    if (EPI) {
        if (w == 0) publish_place(A.place + k.c, base, lane);
        xlocal = __ballot(lane < geo.segs &&
                          !tag_is_local(A.place + static_cast<size_t>(k.t) * geo.segs + lane,
                                        base)) == 0;
        wv = ld_words<W>(a.weight + k.elem);
        res = ld_words<W>(a.residual + k.row);
    }
    for (int i = 0; i < A.reduces; ++i) {
        const uint32_t g = base + static_cast<uint32_t>(i) + 1u;
        const uint32_t p = static_cast<uint32_t>(i + 1) & 1u;
        const size_t pc = static_cast<size_t>(p) * geo.w_max + k.c;
        const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(
            a.slots + static_cast<uint64_t>(p) * geo.slot_elems + chunk_first(geo, k));
        uint32_t *stamp = a.stamps + pc * N;
        const uint32_t *stamp_lane = stamp + (lane < N ? lane : N - 1);
        auto load = [&](Words<W>(&v)[N]) {
#pragma unroll
            for (int r = 0; r < N; ++r)
                v[r] = ld_words_agent_at<W>(rs, off, static_cast<uint32_t>(r) * rank_bytes);
        };
        phase_barrier();
        uint64_t word = 0;  // the previous epoch's exchange word
        if (EPI && i > 0) word = epi_word(a, k, pending.g, lane);
        Words<W> v[N];
        uint32_t st = 0, attempts = 1, first = 0, last = 0;
        uint32_t inj = 0;
        if (INJECT) inj = inject_word(a.inject, a.inject_div, g);
        if (MODE != kOrdered) load(v);
        if (MODE != kNone) st = ld_relaxed(stamp_lane);
        // speculative: the sum runs as the payload arrives, the stamps decide
        // afterwards whether it stands
        Words<W> o;
        if (MODE != kOrdered) o = sum_round<N, W>(v);
        const uint32_t st_first = st;
        if (MODE != kNone) {
            uint32_t m = static_cast<uint32_t>(__ballot(lane < N && st != g));
            first = last = m;
            bool fail = m != 0 || a.forced_retries >= 1;
            // without a table no stamp is late: the loop stays out of the way
            while (INJECT ? fail : __builtin_expect(fail, false)) {
                if (attempts >= a.max_attempts) {
                    if (lane == 0) latch(a.err, kErrRetryBudget, g, k.c, attempts);
                    break;
                }
                if (INJECT && attempts == 1 && m != 0)
                    catch_up<N>(a, k, g, p, late_ranks(__builtin_amdgcn_readfirstlane(inj)), lane,
                                stamp);
                __atomic_signal_fence(__ATOMIC_SEQ_CST);
                if (MODE != kOrdered) load(v);
                st = ld_relaxed(stamp_lane);
                ++attempts;
                m = static_cast<uint32_t>(__ballot(lane < N && st != g));
                last = m;
                fail = m != 0 || attempts <= a.forced_retries;
                // the last load's sum, also of a chunk whose budget runs out
                // (after the loop it would keep the payload registers alive)
                if (MODE != kOrdered && (!fail || attempts >= a.max_attempts))
                    o = sum_round<N, W>(v);
            }
        }
        if (MODE == kOrdered) {
            __atomic_signal_fence(__ATOMIC_SEQ_CST);
            load(v);
            o = sum_round<N, W>(v);
        }
        complete(o);  // every payload load has returned: the slot is free
        if (lane == 0)
            __hip_atomic_store(&done[p][w], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (C == 1 || w == 0) {
            write_log(a, k, g, log_word(attempts, first, last));
            write_stamp_log<N>(a, k, g, lane < N ? lane : N - 1, st_first, st);
            st_flag(a.consumed + pc, g, true);
        }
        const uint64_t ring = static_cast<uint64_t>(i) * A.ring_stride;
        if (!EPI) {
            // lanes past the row's end store the owning lane's bytes again
            st_stream<W>(a.out + ring + k.row, o);
        } else {
            EpiPending<W> cur;
            epi_stage<W>(a, k, g, o, res, lane, k.s * C + w, xlocal, cur);
            if (i > 0) epi_finish<W>(a, k, pending, word, wv, a.y + ring - A.ring_stride, lane);
            pending = cur;
        }
    }
    if (EPI) {
        if (k.lane_ok) st_words<W>(a.residual + k.row, res);
        epi_finish<W>(a, k, pending, epi_word(a, k, pending.g, lane), wv,
                      a.y + static_cast<uint64_t>(A.reduces - 1) * A.ring_stride, lane);
    }
}

// Grid (segs, tokens), C consumer waves and one producer wave; with the
// epilogue (8 * ceil(tokens / 8) * segs) with every workgroup of a token on one
// XCD, as in chain_kernel (workgroups past the last token only arrive on the
// counter). The last workgroup to arrive on the counter advances the epoch base
// for the next step: every wave of a workgroup read it before its first
// barrier.
template <int N, int MODE, bool EPI, bool INJECT, int C>
__global__ __launch_bounds__((C + 1) * kLanes, EPI ? 5 : 8) void step_kernel(ChainArgs A) {
    __shared__ uint32_t done[2][C];
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kLanes);
    const uint32_t base = A.r.ep.base[0];
    int bx = blockIdx.x, by = blockIdx.y;
    if (EPI) {
        const int j = static_cast<int>(blockIdx.x) >> 3;
        bx = j % A.r.geo.segs;
        by = (static_cast<int>(blockIdx.x) & 7) + 8 * (j / A.r.geo.segs);
    }
    if (!EPI || by < A.r.geo.tokens) {
        const Chunk k = chunk_at(A.r.geo, by, bx, lane);
        if (wave == C) {
            step_producer<N, INJECT, C>(A, base, k, lane, done);
            return;
        }
        step_consumer<N, MODE, EPI, INJECT, C>(A, base, k, wave, lane, done);
    }
    if (threadIdx.x == 0) {
        const uint32_t before =
            __hip_atomic_fetch_add(A.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == gridDim.x * gridDim.y - 1u) {
            st_relaxed(A.done, 0u);
            st_relaxed(A.epoch_base, base + A.advance);
        }
    }
}

// ---------------------------------------------------------------------------
// One all-reduce in one launch (the allocation-free call): the phases of
// step_kernel for a single epoch. Wave 1 of a chunk's workgroup plays the
// peers, a barrier follows, wave 0 loads payload and stamps together, sums as
// they arrive and validates. What bounds it: one launch, a round trip for the
// sources and one for the payload. As a producer and a reduction launch the
// call took 10.9 us (N = 8, 16 tokens x 4096, calls back to back from Python),
// 5.0 so, most of it the caller's.
// The arguments up to the source loads lead, to be preloaded into scalar
// registers; the epoch itself is one of them.
template <int N>
__global__ __launch_bounds__(2 * kLanes, 8) void once_kernel(const uint16_t *src,
                                                             int64_t rank_stride, uint16_t *slots,
                                                             uint64_t slot_elems, uint32_t *stamps,
                                                             uint32_t g, int32_t hidden,
                                                             int32_t segs, int32_t w_max,
                                                             OnceArgs a) {
    const int lane = threadIdx.x & (kLanes - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kLanes);
    Geometry geo{};
    geo.hidden = hidden;
    geo.segs = segs;
    const Chunk k = chunk_at(geo, blockIdx.y, blockIdx.x, lane);
    const uint32_t p = g & 1u;
    const size_t pc = static_cast<size_t>(p) * w_max + k.c;
    const uint64_t at = static_cast<uint64_t>(p) * slot_elems + chunk_first(geo, k);
    const uint32_t off = lane_offset(geo, k);
    const uint32_t rank_bytes = static_cast<uint32_t>(slot_elems) * 4u;
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(slots + at);
    uint32_t *stamp = stamps + pc * N;
    V16 v[N];
    if (wave == 1) {
#pragma unroll
        for (int r = 0; r < N; ++r) v[r] = ld16(src + r * rank_stride + k.row);
        const uint32_t prev = ld_relaxed(a.produced + pc), fin = ld_relaxed(a.consumed + pc);
#pragma unroll
        for (int r = 0; r < N; ++r) st16_at(rs, off, static_cast<uint32_t>(r) * rank_bytes, v[r]);
        if (lane == 0 && prev != fin) latch(a.err, kErrWaw, g, k.c, prev);
        // the stamps follow the payload
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane < N) st_flag(stamp + lane, g, true);
        if (lane == 0) st_flag(a.produced + pc, g, true);
        phase_barrier();
        return;
    }
    phase_barrier();
    uint32_t attempts = 0, m = 0, first = 0;
    V16 o;
    while (true) {
#pragma unroll
        for (int r = 0; r < N; ++r)
            v[r] = ld16_agent_at(rs, off, static_cast<uint32_t>(r) * rank_bytes);
        const uint32_t st = ld_relaxed(stamp + (lane < N ? lane : N - 1));
        o = sum_round<N, 4>(v);
        m = static_cast<uint32_t>(__ballot(lane < N && st != g));
        if (attempts++ == 0) first = m;
        // a stale stamp can only come from a call that overlaps this one
        if (m == 0) break;
        if (attempts >= a.max_attempts) {
            if (lane == 0) latch(a.err, kErrRetryBudget, g, k.c, attempts);
            break;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    if (lane == 0) {
        a.log[k.c] = log_word(attempts, first, m);
        a.consumed[pc] = g;
    }
    if (k.lane_ok) st16_stream(a.out + k.row, o);
}

__global__ void advance_kernel(uint32_t *base, uint32_t step) {
    if (threadIdx.x == 0) base[0] += step;
}

__global__ void set_base_kernel(uint32_t *base, uint32_t value) {
    if (threadIdx.x == 0) base[0] = value;
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t value, uint64_t count) {
    for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < count;
         i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
        p[i] = value;
}

template <int N, int MODE>
hipError_t launch_reduce_nm(const ReduceArgs &a, const ProduceArgs *pa, bool epi, dim3 grid,
                            dim3 block, hipStream_t s) {
    const ProduceArgs none{};
    int lg = 0;
    while ((kLanes << lg) < static_cast<int>(block.x)) ++lg;
    if ((kLanes << lg) != static_cast<int>(block.x) || lg > 4) return hipErrorInvalidValue;
    if (a.geo.hidden < 1 || a.geo.hidden > 0x10000 || a.geo.segs < 1 || a.geo.segs > 0xFF ||
        a.ep.parity > 1)
        return hipErrorInvalidValue;
    // the producer plane shares the leading arguments (one handle's slots,
    // stamps, epoch and geometry)
    if (pa && (pa->ep.base != a.ep.base || pa->slots != a.slots || pa->stamps != a.stamps ||
               pa->geo.hidden != a.geo.hidden || pa->geo.w_max != a.geo.w_max ||
               pa->geo.slot_elems != a.geo.slot_elems))
        return hipErrorInvalidValue;
    const uint32_t shape = static_cast<uint32_t>(a.geo.hidden) |
                           (static_cast<uint32_t>(a.geo.segs) << 17) | (a.ep.parity << 25) |
                           (static_cast<uint32_t>(lg) << 26);
    const uint32_t w_max = static_cast<uint32_t>(a.geo.w_max);
#define SIFAR_REDUCE_LAUNCH(EPI_, FUSED_, PA_)                                                   \
    hipLaunchKernelGGL((reduce_kernel<N, MODE, EPI_, FUSED_>), grid, block, 0, s, a.ep.base,   \
                       a.slots, a.stamps, a.geo.slot_elems, shape, w_max, a.ep.off, a, PA_)
    if (pa) {
        grid.z = 2;
        if (epi)
            SIFAR_REDUCE_LAUNCH(true, true, *pa);
        else
            SIFAR_REDUCE_LAUNCH(false, true, *pa);
    } else {
        if (epi)
            SIFAR_REDUCE_LAUNCH(true, false, none);
        else
            SIFAR_REDUCE_LAUNCH(false, false, none);
    }
#undef SIFAR_REDUCE_LAUNCH
    return hipGetLastError();
}

template <int N>
hipError_t launch_reduce_n(const ReduceArgs &a, const ProduceArgs *pa, int mode, bool epi,
                           dim3 grid, dim3 block, hipStream_t s) {
    switch (mode) {
        case kSpec: return launch_reduce_nm<N, kSpec>(a, pa, epi, grid, block, s);
        case kOrdered: return launch_reduce_nm<N, kOrdered>(a, pa, epi, grid, block, s);
        case kNone: return launch_reduce_nm<N, kNone>(a, pa, epi, grid, block, s);
    }
    return hipErrorInvalidValue;
}

// With the epilogue the consumer sets the register count, so only the plain
// kernel comes in both producer forms.
template <int N, int MODE>
const void *chain_fn(bool epi, bool prefetch) {
    if (epi) return reinterpret_cast<const void *>(chain_kernel<N, MODE, true, true>);
    return prefetch ? reinterpret_cast<const void *>(chain_kernel<N, MODE, false, true>)
                    : reinterpret_cast<const void *>(chain_kernel<N, MODE, false, false>);
}

// Persistent steps validate before they load: ORDERED only.
template <int N>
const void *chain_fn_n(int mode, bool epi, bool prefetch) {
    return mode == kOrdered ? chain_fn<N, kOrdered>(epi, prefetch) : nullptr;
}

const void *chain_fn_any(int nranks, int mode, bool epi, bool prefetch) {
    switch (nranks) {
        case 1: return chain_fn_n<1>(mode, epi, prefetch);
        case 2: return chain_fn_n<2>(mode, epi, prefetch);
        case 3: return chain_fn_n<3>(mode, epi, prefetch);
        case 4: return chain_fn_n<4>(mode, epi, prefetch);
        case 5: return chain_fn_n<5>(mode, epi, prefetch);
        case 6: return chain_fn_n<6>(mode, epi, prefetch);
        case 7: return chain_fn_n<7>(mode, epi, prefetch);
        case 8: return chain_fn_n<8>(mode, epi, prefetch);
    }
    return nullptr;
}

// `inject`: the kernel that knows the injection table and the stage (one
// consumer wave). NONE validates nothing, so it has no injection.
template <int N, int MODE, bool EPI>
const void *step_fn(bool inject, int consumers) {
    if (inject) {
        if (MODE == kNone || consumers != 1) return nullptr;
        return reinterpret_cast<const void *>(
            step_kernel<N, MODE == kNone ? kSpec : MODE, EPI, true, 1>);
    }
    switch (consumers) {
        case 1: return reinterpret_cast<const void *>(step_kernel<N, MODE, EPI, false, 1>);
        case kStepConsumers:
            return reinterpret_cast<const void *>(step_kernel<N, MODE, EPI, false, kStepConsumers>);
    }
    return nullptr;
}

template <int N>
const void *step_fn_n(int mode, bool epi, bool inject, int consumers) {
    switch (mode) {
        case kSpec:
            return epi ? step_fn<N, kSpec, true>(inject, consumers)
                       : step_fn<N, kSpec, false>(inject, consumers);
        case kOrdered:
            return epi ? step_fn<N, kOrdered, true>(inject, consumers)
                       : step_fn<N, kOrdered, false>(inject, consumers);
        case kNone:
            return epi ? step_fn<N, kNone, true>(inject, consumers)
                       : step_fn<N, kNone, false>(inject, consumers);
    }
    return nullptr;
}

const void *step_fn_any(int nranks, int mode, bool epi, bool inject, int consumers) {
    switch (nranks) {
        case 1: return step_fn_n<1>(mode, epi, inject, consumers);
        case 2: return step_fn_n<2>(mode, epi, inject, consumers);
        case 3: return step_fn_n<3>(mode, epi, inject, consumers);
        case 4: return step_fn_n<4>(mode, epi, inject, consumers);
        case 5: return step_fn_n<5>(mode, epi, inject, consumers);
        case 6: return step_fn_n<6>(mode, epi, inject, consumers);
        case 7: return step_fn_n<7>(mode, epi, inject, consumers);
        case 8: return step_fn_n<8>(mode, epi, inject, consumers);
    }
    return nullptr;
}

template <int N, int MODE>
const void *reduce_fn(bool epi) {
    // the fused variant is the larger of the two: use it for occupancy
    return epi ? reinterpret_cast<const void *>(reduce_kernel<N, MODE, true, true>)
               : reinterpret_cast<const void *>(reduce_kernel<N, MODE, false, true>);
}

template <int N>
const void *reduce_fn_n(int mode, bool epi) {
    switch (mode) {
        case kSpec: return reduce_fn<N, kSpec>(epi);
        case kOrdered: return reduce_fn<N, kOrdered>(epi);
        case kNone: return reduce_fn<N, kNone>(epi);
    }
    return nullptr;
}

const void *reduce_fn_any(int nranks, int mode, bool epi) {
    switch (nranks) {
        case 1: return reduce_fn_n<1>(mode, epi);
        case 2: return reduce_fn_n<2>(mode, epi);
        case 3: return reduce_fn_n<3>(mode, epi);
        case 4: return reduce_fn_n<4>(mode, epi);
        case 5: return reduce_fn_n<5>(mode, epi);
        case 6: return reduce_fn_n<6>(mode, epi);
        case 7: return reduce_fn_n<7>(mode, epi);
        case 8: return reduce_fn_n<8>(mode, epi);
    }
    return nullptr;
}

int resident_groups(const void *fn, int threads) {
    if (!fn) return 0;
    int per_cu = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0) != hipSuccess)
        return 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return per_cu * cus;
}

}  // namespace

hipError_t launch_produce(const ProduceArgs &a, int waves_per_group, hipStream_t s) {
    const dim3 grid(static_cast<uint32_t>((a.geo.segs + waves_per_group - 1) / waves_per_group),
                    static_cast<uint32_t>(a.geo.tokens));
    const dim3 block(waves_per_group * kLanes);
    switch (a.geo.nranks) {
        case 1: hipLaunchKernelGGL(produce_kernel<1>, grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL(produce_kernel<2>, grid, block, 0, s, a); break;
        case 3: hipLaunchKernelGGL(produce_kernel<3>, grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL(produce_kernel<4>, grid, block, 0, s, a); break;
        case 5: hipLaunchKernelGGL(produce_kernel<5>, grid, block, 0, s, a); break;
        case 6: hipLaunchKernelGGL(produce_kernel<6>, grid, block, 0, s, a); break;
        case 7: hipLaunchKernelGGL(produce_kernel<7>, grid, block, 0, s, a); break;
        case 8: hipLaunchKernelGGL(produce_kernel<8>, grid, block, 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs &a, const ProduceArgs *next, int mode, bool epilogue,
                         int waves_per_group, hipStream_t s) {
    const dim3 block(waves_per_group * kLanes);
    const dim3 grid(static_cast<uint32_t>((a.geo.segs + waves_per_group - 1) / waves_per_group),
                    static_cast<uint32_t>(a.geo.tokens));
    if (next && (next->geo.segs != a.geo.segs || next->geo.tokens != a.geo.tokens))
        return hipErrorInvalidValue;
    switch (a.geo.nranks) {
        case 1: return launch_reduce_n<1>(a, next, mode, epilogue, grid, block, s);
        case 2: return launch_reduce_n<2>(a, next, mode, epilogue, grid, block, s);
        case 3: return launch_reduce_n<3>(a, next, mode, epilogue, grid, block, s);
        case 4: return launch_reduce_n<4>(a, next, mode, epilogue, grid, block, s);
        case 5: return launch_reduce_n<5>(a, next, mode, epilogue, grid, block, s);
        case 6: return launch_reduce_n<6>(a, next, mode, epilogue, grid, block, s);
        case 7: return launch_reduce_n<7>(a, next, mode, epilogue, grid, block, s);
        case 8: return launch_reduce_n<8>(a, next, mode, epilogue, grid, block, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_chain(const ChainArgs &a, int mode, bool epilogue, bool prefetch, hipStream_t s) {
    const void *fn = chain_fn_any(a.r.geo.nranks, mode, epilogue, prefetch);
    if (!fn) return hipErrorInvalidValue;
    if (a.r.geo.segs != a.p.geo.segs || a.r.geo.tokens != a.p.geo.tokens)
        return hipErrorInvalidValue;
    const uint32_t segs = static_cast<uint32_t>(a.r.geo.segs);
    const uint32_t t8 = (static_cast<uint32_t>(a.r.geo.tokens) + 7u) / 8u;
    if (epilogue && (a.r.geo.segs > kLanes || a.r.groups_per_token != a.r.geo.segs))
        return hipErrorInvalidValue;
    // the slots are addressed at 32-bit offsets from rank 0's (payload loads,
    // slot stores); co-residency keeps a step far below that (at most 4096
    // chunks: under 64 MiB of slots)
    if (!step_offsets_fit(a.r.geo.nranks, a.r.geo.slot_elems)) return hipErrorInvalidValue;
    const dim3 grid = epilogue ? dim3(8u * t8 * segs, 1, 2)
                               : dim3(segs, static_cast<uint32_t>(plane_rows(a.r.geo.tokens, segs)), 2);
    void *args[] = {const_cast<ChainArgs *>(&a)};
    return hipLaunchKernel(fn, grid, dim3(kLanes), args, 0, s);
}

hipError_t launch_once(const Geometry &geo, uint32_t g, const uint16_t *src, int64_t rank_stride,
                       uint16_t *slots, uint32_t *stamps, const OnceArgs &a, hipStream_t s) {
    if (!step_offsets_fit(geo.nranks, geo.slot_elems)) return hipErrorInvalidValue;
    const dim3 grid(static_cast<uint32_t>(geo.segs), static_cast<uint32_t>(geo.tokens));
#define SIFAR_ONCE(N_)                                                                             \
    case N_:                                                                                       \
        hipLaunchKernelGGL(once_kernel<N_>, grid, dim3(2 * kLanes), 0, s, src, rank_stride, slots, \
                           geo.slot_elems, stamps, g, geo.hidden, geo.segs, geo.w_max, a);         \
        break
    switch (geo.nranks) {
        SIFAR_ONCE(1);
        SIFAR_ONCE(2);
        SIFAR_ONCE(3);
        SIFAR_ONCE(4);
        SIFAR_ONCE(5);
        SIFAR_ONCE(6);
        SIFAR_ONCE(7);
        SIFAR_ONCE(8);
        default: return hipErrorInvalidValue;
    }
#undef SIFAR_ONCE
    return hipGetLastError();
}

hipError_t launch_step(const ChainArgs &a, int mode, bool epilogue, int consumers,
                       hipStream_t s) {
    const void *fn = step_fn_any(a.r.geo.nranks, mode, epilogue, a.p.stage != nullptr, consumers);
    if (epilogue && (a.r.geo.segs * consumers > kLanes ||
                     a.r.groups_per_token != a.r.geo.segs * consumers))
        return hipErrorInvalidValue;
    if (!fn || a.parity_mask != 1u || !a.r.stamp_log || (a.p.inject && !a.p.stage))
        return hipErrorInvalidValue;
    // slots and sources are addressed at 32-bit offsets from rank 0's
    if (!step_offsets_fit(a.r.geo.nranks, a.r.geo.slot_elems) ||
        !source_offsets_fit(a.r.geo.nranks, a.p.rank_stride))
        return hipErrorInvalidValue;
    const uint32_t segs = static_cast<uint32_t>(a.r.geo.segs);
    const uint32_t tokens = static_cast<uint32_t>(a.r.geo.tokens);
    const dim3 grid = epilogue ? dim3((tokens + 7u) / 8u * 8u * segs) : dim3(segs, tokens);
    void *args[] = {const_cast<ChainArgs *>(&a)};
    return hipLaunchKernel(fn, grid, dim3((consumers + 1) * kLanes), args, 0, s);
}

int max_active_split_step_groups(int nranks, int mode, bool epilogue) {
    return resident_groups(step_fn_any(nranks, mode, epilogue, false, kStepConsumers),
                           (kStepConsumers + 1) * kLanes);
}

int max_active_step_groups(int nranks, int mode, bool epilogue) {
    const int lean = resident_groups(step_fn_any(nranks, mode, epilogue, false, 1), 2 * kLanes);
    const void *fn = step_fn_any(nranks, mode, epilogue, true, 1);
    const int full = fn ? resident_groups(fn, 2 * kLanes) : lean;
    return full < lean ? full : lean;
}

int max_active_groups(int nranks, int mode, bool epilogue, int waves_per_group) {
    return resident_groups(reduce_fn_any(nranks, mode, epilogue), waves_per_group * kLanes);
}

int max_active_chain_waves(int nranks, int mode, bool epilogue, bool prefetch) {
    return resident_groups(chain_fn_any(nranks, mode, epilogue, prefetch), kLanes);
}

hipError_t launch_advance(uint32_t *epoch_base, uint32_t step, hipStream_t s) {
    hipLaunchKernelGGL(advance_kernel, dim3(1), dim3(kLanes), 0, s, epoch_base, step);
    return hipGetLastError();
}

hipError_t launch_set_base(uint32_t *epoch_base, uint32_t value, hipStream_t s) {
    hipLaunchKernelGGL(set_base_kernel, dim3(1), dim3(kLanes), 0, s, epoch_base, value);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t value, uint64_t count, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const uint64_t blocks64 = (count + 255) / 256;
    const dim3 grid(static_cast<uint32_t>(blocks64 < 4096 ? blocks64 : 4096));
    hipLaunchKernelGGL(fill_u32_kernel, grid, dim3(256), 0, s, p, value, count);
    return hipGetLastError();
}

}  // namespace sifar
