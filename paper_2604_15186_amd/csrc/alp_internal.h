// Internal declarations shared by the ABI layer (alp_api.hip) and the gfx950 kernels
// (alp_kernels.hip).  Not installed; the public interface is include/alp.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "alp.h"

namespace alp {

// Share-unit value stored for an option that cannot be used at the query's target (not
// deployable, weights do not fit, or the replica load exceeds saturation).  Real share units
// are at most 64 * 16 * 16 = 16384 per LLM and 131072 per candidate, budgets are clamped
// below the sentinel, so any candidate containing such an option fails the budget test.
constexpr uint32_t kSentinelUnits = 1u << 24;
constexpr uint32_t kCapacityMax = kSentinelUnits - 1;
constexpr uint32_t kNoLatency = 0xFFFFFFFFu;

// Search-space shape passed by value to kernels.  mul_O and mul_D are the multipliers of
// div_by(): ceil(2^32 / O) and ceil(2^32 / D), 0 for a divisor of 1.  The tensor-parallel
// degrees (at most 64) and GPU shares (at most 16 units) are bytes of tp8 and fq8 (byte i the
// i-th value), so that a lane picks its own by a shift: a by-value array indexed differently
// by different lanes is read from the kernel-argument memory, one slow round trip.
struct SpaceDev {
    uint32_t M, n_tp, n_fq, D, K, Q, O;
    uint32_t mul_O, mul_D;
    uint64_t tp8, fq8;
    __host__ __device__ uint32_t tp(uint32_t i) const { return (uint32_t)(tp8 >> (8 * i)) & 0xFFu; }
    __host__ __device__ uint32_t fq(uint32_t j) const { return (uint32_t)(fq8 >> (8 * j)) & 0xFFu; }
};

// The multiplier div_by() takes for divisor v (1 <= v < 2^32).
__host__ __device__ inline uint32_t div_multiplier(uint32_t v)
{
    return v > 1 ? (uint32_t)((UINT64_C(0xFFFFFFFF) + v) / v) : 0u;
}

// floor(a / v) for a * v < 2^32, given mul = div_multiplier(v): with mul = (2^32 + e) / v,
// 0 <= e < v, a * mul / 2^32 = a / v + a e / (v 2^32) and the added part is below 1 / v, less
// than the distance from a / v to the next integer.
__host__ __device__ inline uint32_t div_by(uint32_t a, uint32_t mul)
{
    return mul ? (uint32_t)(((uint64_t)a * mul) >> 32) : a;
}

// Device copies of the profile tables of all instances (layouts as in alp_load_profiles).
struct TablesDev {
    const uint64_t *W;
    const uint32_t *n;
    const uint32_t *p;
    const uint8_t *allowed;
    const uint32_t *rate;
    const uint32_t *lat;
    uint64_t H;
};

// Per-item query: device arrays for batches, or by-value scalars for a single query.
// The three arrays are set together or not at all.
struct QueryDev {
    const uint32_t *inst;       // instance of item i, or nullptr -> inst1
    const uint32_t *capacity;   // share-unit capacity Q*G of item i (clamped), or nullptr -> cap1
    const uint32_t *lambda;     // target rate of item i, or nullptr -> lambda1
    uint32_t inst1, cap1, lambda1;
};

// Records per item of the inner-LLM table: options rounded up to a multiple of 16.
__host__ __device__ inline uint32_t inner_stride(uint32_t O) { return (O + 15u) & ~15u; }
// Records per item of the pair table (LLMs M-3 and M-2 folded into one inner LLM of O^2
// options), padded to 16.
__host__ __device__ inline uint32_t pair_stride(uint32_t O) { return (O * O + 15u) & ~15u; }

// Per-block winner of a scan: lexicographic (L, x) minimum; L = kNoLatency if none.
struct Winner {
    uint32_t L;
    uint32_t pad;
    uint64_t x;
};

// The scan kernels write alp_result_t as six 64-bit words in this field order.
static_assert(sizeof(alp_result_t) == 48, "alp_result_t layout");
static_assert(offsetof(alp_result_t, latency_us) == 8 && offsetof(alp_result_t, throughput_milli) == 12 &&
                  offsetof(alp_result_t, gpu_units) == 16 && offsetof(alp_result_t, status) == 20 &&
                  offsetof(alp_result_t, tp) == 24 && offsetof(alp_result_t, frac_units) == 32 &&
                  offsetof(alp_result_t, replicas) == 40,
              "alp_result_t layout");

// What the last block of an item needs to produce the item's result.
struct FinishArgs {
    SpaceDev sp;
    const uint2 *ext;          // per-option (tau, u | flags) of the query
    uint32_t *done;            // per-item finished-block counter, zeroed by the option-term kernel
    uint32_t *best;            // per-item smallest block latency seen so far (atomic minimum),
                               // kNoLatency from the option-term kernel
    alp_result_t *out;         // per-item results (device-visible, may be mapped host memory)
    const uint32_t *invalid;   // per-item: nonzero = the query was rejected (result EINVAL);
                               // nullptr = every query valid
    // A search of one item whose caller waits for its record in host memory: once the record is
    // written, seq is stored to *signal (mapped host memory) with a release at system scope, so
    // a host that reads seq there also reads the whole record.  nullptr: no signal.
    uint32_t *signal = nullptr;
    uint32_t seq = 0;
};

// Tiles and scales of the packed scan (alp_packed.hip).  Share units are counted in multiples of
// the greatest common divisor of the space's shares (mul_unit divides by it).
struct PackedPlan {
    uint32_t S;                // above every rank of the inner LLM's usable options
    uint32_t U;                // most units a deployable option uses
    uint32_t mul_unit, mul_fq; // multipliers of div_by() for that divisor and the share count
    uint32_t inv_O;            // floor((2^32 - 1) / O)
    uint32_t wide_index;       // lanes' indices (rows * E of them) need more than 32 bits
    uint32_t wide;             // (U + 1) * S needs the unsigned form
    uint32_t E, chunks;        // lane pairs, and chunks of 128 * slots of them
    uint32_t tiles, tiles_per_block;   // rows_per_block = 0: tiles of an item, and of a block
    uint64_t rows, rows_per_block;     // rows_per_block > 0: a block owns whole rows
};

// Launch geometry of one scan.
struct ScanGeometry {
    uint32_t variant;          // 1: row-minimum, 2: thread-per-candidate, 3: exact-tracking lanes
    uint32_t threads;          // per block
    uint32_t blocks_per_item;
    uint64_t rows;             // variants 1, 3: rows of O prefixes per item (variant 1: sub-rows,
                               // rows times chunks)
    uint64_t rows_per_wave;    // variants 1, 3
    uint32_t chunks;           // variant 1: ranges of the inner LLM's records per row
    uint32_t dynamic;          // variant 1: sub-rows handed out within each block (1) or fixed
                               // per wave (0, requires chunks == 1)
    uint64_t per_thread;       // variant 2: candidates per thread
    uint32_t slots;            // variants 1, 3: options of the last LLM per lane (1, 2, 4, 8)
    uint32_t pair;             // variant 1: the inner table is the pair table (rows fix M - 3
                               // digits, O^2 records each)
    uint32_t fused;            // variant 1: one launch -- every block computes its item's option
                               // terms itself, and the item's winner is one 64-bit word (spaces of
                               // fewer than 2^32 candidates, never with the pair table)
    uint32_t use_packed;       // the packed scan instead (slots: registers of two pairs per lane)
    PackedPlan packed;
};

// Queries of a search batch given in device memory, prepared by the option-term kernel: item i
// searches instance inst[i] (i when inst is nullptr; one >= B is rejected and searched as
// instance 0), capacity min(units_per_gpu * budget[i], kCapacityMax), target target[i].  The
// kernel writes the prepared arrays (the QueryDev the scan reads) and the rejection flags.
struct RawQueries {
    const uint32_t *inst, *budget, *target;
    uint32_t B, units_per_gpu;
    uint32_t *q_inst, *q_cap, *q_lambda, *invalid;
};

// The one-launch form of the scan (ScanGeometry::fused): each block computes the option terms
// of its item from the tables into its own region of device memory and reads them back through
// the scalar cache; the item's best candidate so far is the word best[item] = ~(L << 32 | x)
// (x < 2^32), raised by an atomic maximum, 0 for none; done[item] counts finished blocks.  The
// last block of an item resets both words to 0, so they are 0 between launches (the host zeroes
// them when it allocates them).
struct FusedArgs {
    TablesDev tb;
    RawQueries raw;            // device queries when raw.budget is set (the QueryDev otherwise)
    uint2 *regions;            // per block: M * O option records, then inner_stride(O) records
    uint32_t region;           // records per block region
    uint32_t *done;            // per item: finished block groups
    uint32_t *group_done;      // per item and group of kFusedGroup blocks: finished blocks
    unsigned long long *best;
    unsigned long long *slots; // packed scan: per block, its lowest (latency, lanes' index)
};
// count_block(): blocks counted together, and the distance of its counters in 32-bit words (an
// item has one for its groups, then one per group).
constexpr uint32_t kGroupBlocks = 16, kCounterLine = 32;
__host__ __device__ inline uint64_t block_counter_words(uint64_t items, uint32_t blocks_per_item)
{
    return items * (1 + (blocks_per_item + kGroupBlocks - 1) / kGroupBlocks) * kCounterLine;
}
// Blocks of an item counted together before the item's count (two-level counting, so that at
// most this many blocks update one counter word).
constexpr uint32_t kFusedGroup = 64;

// What the option-term kernel resets for the scan that follows it: per item, the finished-block
// counter (done = 0) and the smallest block latency (best = kNoLatency, if best is set); every
// block winner slot (winners[0..n_winners) = no candidate).
struct ScanReset {
    uint32_t *done = nullptr;
    uint32_t *best = nullptr;
    Winner *winners = nullptr;
    uint64_t n_winners = 0;
};

hipError_t launch_option_terms(const SpaceDev &sp, const TablesDev &tb, const QueryDev &q,
                               uint32_t count, uint2 *rec, uint2 *ext, uint2 *inner,
                               const ScanReset &reset, hipStream_t st,
                               const RawQueries *raw = nullptr,
                               hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr);
// Pair table of count items: pair[item][j3 * O + j2] = (c of LLM M-3 option j3 + c of LLM M-2
// option j2, Q*G - both share units), from the option-term kernel's rec and inner tables;
// padding records never fit.
hipError_t launch_pair_terms(const SpaceDev &sp, uint32_t count, const uint2 *rec,
                             const uint2 *inner, uint2 *pair, hipStream_t st);
// fz: the one-launch form's arguments (g.fused), else nullptr.
hipError_t launch_scan(const SpaceDev &sp, const QueryDev &q, uint32_t count, const uint2 *rec,
                       const uint2 *inner, const ScanGeometry &g, Winner *winners,
                       const FinishArgs &fa, hipStream_t st, hipEvent_t t0 = nullptr,
                       hipEvent_t t1 = nullptr, const FusedArgs *fz = nullptr);
// Dynamic LDS of a one-launch scan block: the item's profile curves (for every (LLM, tp,
// share): rate padded to ALP_MAX_POINTS points, then -- after all rates -- lat, K points) and
// their deployability flags ...
__host__ __device__ inline size_t fused_lds_curves(const SpaceDev &sp)
{
    return (size_t)sp.M * sp.n_tp * sp.n_fq;
}
__host__ __device__ inline size_t fused_lds_lat_offset(const SpaceDev &sp)
{
    return fused_lds_curves(sp) * ALP_MAX_POINTS * sizeof(uint32_t);
}
__host__ __device__ inline size_t fused_lds_deploy_offset(const SpaceDev &sp)
{
    return fused_lds_lat_offset(sp) + fused_lds_curves(sp) * sp.K * sizeof(uint32_t);
}
// ... followed by the inner LLM's records (inner_stride(O) of them), 8-byte aligned.
__host__ __device__ inline size_t fused_lds_inner_offset(const SpaceDev &sp)
{
    return (fused_lds_deploy_offset(sp) + fused_lds_curves(sp) + 7) & ~(size_t)7;
}
// ... then every option's (tau, share units) for the result record.
__host__ __device__ inline size_t fused_lds_ext_offset(const SpaceDev &sp)
{
    return fused_lds_inner_offset(sp) + (size_t)inner_stride(sp.O) * 8;
}
__host__ __device__ inline size_t fused_lds_bytes(const SpaceDev &sp)
{
    return fused_lds_ext_offset(sp) + (size_t)sp.M * sp.O * 8;
}
// Records per block region of the one-launch form.
__host__ __device__ inline uint32_t fused_region(uint32_t M, uint32_t O)
{
    return (M * O + inner_stride(O) + 7u) & ~7u;    // 64-byte multiple
}
// Dynamic LDS of a packed scan block: the curves and deployability flags as above, the inner
// LLM's terms (inner_stride(O) words), every option's (tau, share units) and (term, units), and
// the term of each rank.
__host__ __device__ inline size_t packed_lds_key_offset(const SpaceDev &sp)
{
    return (fused_lds_deploy_offset(sp) + fused_lds_curves(sp) + 15) & ~(size_t)15;
}
__host__ __device__ inline size_t packed_lds_ext_offset(const SpaceDev &sp)
{
    return packed_lds_key_offset(sp) + (size_t)inner_stride(sp.O) * 4;
}
__host__ __device__ inline size_t packed_lds_bytes(const SpaceDev &sp, uint32_t S)
{
    return packed_lds_ext_offset(sp) + (size_t)sp.M * sp.O * 16 + ((size_t)S + 1) * 4;
}
hipError_t launch_packed(const SpaceDev &sp, const QueryDev &q, uint32_t count,
                         const ScanGeometry &g, const FinishArgs &fa, const FusedArgs &fz,
                         hipStream_t st, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr);
hipError_t launch_eval(const SpaceDev &sp, uint32_t capacity, const uint2 *rec, const uint2 *ext,
                       const uint64_t *idx, uint64_t count, alp_eval_t *out, hipStream_t st);
hipError_t launch_tmax(const SpaceDev &sp, const TablesDev &tb, const QueryDev &q, uint32_t count,
                       uint32_t *out, hipStream_t st);

// Budget split over W workflows from their per-budget search results (res[w * (G + 1) + g]),
// see alp_allocate_workflows.  dp: device scratch of (W + 1) * (G + 1) uint64 followed by
// 2 * W * (G + 1) uint32.  Writes *plan and gpus[0..W).
hipError_t launch_allocate(const alp_result_t *res, uint32_t W, uint32_t G, uint32_t policy,
                           uint64_t *dp, alp_plan_t *plan, uint32_t *gpus, hipStream_t st);

// The paper's pruned search for count items of at most F_max units (see alp_search_pruned), after
// the option-term kernel (rec, ext).  table: count * pruned_table_entries() entries of device
// memory (0: the blocks build it in LDS); pruned_blocks_per_item() blocks per item, three words of
// slots for each, and block_counter_words() counters, 0 between launches.  Records table_done (if
// given) before the enumeration.  Writes out[0..count).
uint64_t pruned_table_entries(const SpaceDev &sp, uint32_t F_max, uint32_t flags);
uint32_t pruned_blocks_per_item(const SpaceDev &sp, uint32_t F_max, uint32_t flags,
                                uint32_t count);
hipError_t launch_pruned(const SpaceDev &sp, const TablesDev &tb, const QueryDev &q, uint32_t count,
                         uint32_t F_max, uint32_t flags, const uint2 *rec, uint64_t *table,
                         uint32_t blocks_per_item, uint64_t *slots, uint32_t *counters,
                         const uint2 *ext, alp_pruned_t *out, hipStream_t st,
                         hipEvent_t table_done);

static_assert(sizeof(alp_stats_t) == 32 && offsetof(alp_stats_t, calls) == 8 &&
                  offsetof(alp_stats_t, active_us) == 24,
              "alp_stats_t layout");
static_assert(sizeof(alp_pruned_t) == 64 && offsetof(alp_pruned_t, fraction_vectors) == 48 &&
                  offsetof(alp_pruned_t, unpruned_vectors) == 56,
              "alp_pruned_t layout");

// Workflow statistics (see alp_trace_stats).  totals: kStatsTotalsWords + kStatsTailWords words:
// kStatsCopies copies of the per-LLM sums (and the direct sort's measures), kStatsCopyStride words
// apart (trace r adds to copy r mod kStatsCopies, so that thousands of traces do not queue on the
// same atomic words), then the status flags and the count of long traces (the low and high half of
// one word), the length of the work list and the count of finished slots (of the next), and
// kStatsSlots 32-bit counters of finished blocks.  They must be zero when the kernels start; the
// last block leaves them zero, so zero_first is needed only for fresh memory or after a failed
// launch.
constexpr uint32_t kStatsCopies = 64;
constexpr uint32_t kStatsCopyStride = 32;                 // >= 3 * ALP_MAX_LLMS + 2, 256 B apart
constexpr uint32_t kStatsTotalsWords = kStatsCopies * kStatsCopyStride;
constexpr uint32_t kStatsSlots = 64;
constexpr uint32_t kStatsTailWords = 2 + kStatsSlots / 2;
constexpr uint32_t kStatsShortMax = 2048;                 // calls of a trace swept or sorted in LDS
struct StatsTail {
    uint32_t flags;                   // status bits (see alp_trace_stats)
    uint32_t listed;                  // traces the sweep left to the sort pass
    uint32_t longs;                   // traces beyond kStatsShortMax, left to a second launch
    uint32_t longest;                 // longest trace above 512 calls that the direct sort saw or
                                      // the sweep listed (0: none)
    uint32_t in_order;                // direct sort: traces whose calls came in end order (empty
                                      // ones are)
    uint32_t pad[2];
    uint32_t seq;                     // the launch's seq, stored last
};
static_assert(sizeof(StatsTail) == sizeof(alp_stats_t), "the tail takes one record's place");
// What a launch does with the traces of at most lds_cap calls: sweeps those in end order and lists
// the others in work (R entries) for the sort pass; sorts every one directly (group sizes up to
// max_short calls; longer ones are listed); or leaves them (an earlier launch summed them, and only
// the long traces are to come).
enum StatsOrder { kStatsSweep, kStatsDirect, kStatsLongOnly };
struct StatsLaunch {
    StatsOrder order;
    uint32_t M, R;
    const uint64_t *offsets;
    const uint32_t *llm;
    const uint64_t *start, *end;
    uint32_t lds_cap;                 // a power of two, 256..kStatsShortMax
    uint32_t max_short;
    uint64_t num_calls;               // entries of the call arrays
    bool planned;                     // the host has read the offsets; otherwise the kernels check
                                      // them (against num_calls) and count the long traces
    uint32_t num_long;                // planned: traces beyond lds_cap, long_traces[], sorted in
    const uint32_t *long_traces;      // scratch, trace k at 2 * long_base[k] words
    const uint64_t *long_base;        // (2 * pow2(length) words each)
    uint64_t *scratch, *totals;
    uint32_t *work;
    bool zero_first;
    alp_stats_t *out;                 // M records, then the StatsTail at out[ALP_MAX_LLMS]
    uint32_t seq;
};
hipError_t launch_trace_stats(const StatsLaunch &l, hipStream_t st);

// One allocation to place: budget, LLM count, whether the search found it, per-LLM choices,
// and the index of its output record.
struct PlaceIn {
    uint8_t gpus, llms, feasible, pad;
    uint8_t tp[ALP_MAX_LLMS], q[ALP_MAX_LLMS], d[ALP_MAX_LLMS];
    uint32_t dst;
};

// Placement (see alp_place); Q share units per GPU.  in[0..small) have budgets of at most 16
// GPUs (placed four to a wave), in[small..small + large) the others (one to a wave); each
// writes record in[i].dst of out: an alp_placement_t cut to its first `slots` slots (a multiple of
// 8, at least every allocation's replicas).
hipError_t launch_place(uint32_t Q, uint32_t slots, uint32_t small, uint32_t large,
                        const PlaceIn *in, uint32_t *out, hipStream_t st);

static_assert(sizeof(alp_placement_t) == 272 && offsetof(alp_placement_t, slot) == 16,
              "alp_placement_t layout");

// Device address of the fixed scratch array of alp_search_batch_async_noalloc on `device`, which
// must be the current device.  Looked up once per device; later calls return the kept address.
hipError_t static_scratch_address(int device, void **ptr);

// Resident blocks per CU of the scan kernels at a given block size (occupancy query).
int scan_blocks_per_cu(uint32_t variant, uint32_t slots, uint32_t threads, const SpaceDev &sp);

}  // namespace alp
