// gfx950 kernels of the paper's own pruned allocation search (Scepsy, arXiv 2604.15186,
// Section 5, steps 1-3), measured against the exhaustive search of alp_kernels.hip.
//
//   Step 1  every LLM m gets f_m units of 1/Q GPU, sum f_m = Q*G; with the ordering flag no LLM
//           gets more units than one of higher profiled latency ratio before it, with the
//           minimum-fraction flag every LLM gets at least the units that hold its weights and
//           at most Q*G minus the lower bounds of the LLMs after it.
//   Step 2  the fractions are packed contiguously, highest latency ratio first.
//   Step 3  an option (tp, q, d) is admissible for an LLM iff tp*q*d equals its fraction and
//           d replicas of tp ranks (q units each, the ranks of a replica on distinct GPUs) fit
//           its packed GPUs.
//
// Kernels:
//   pruned_scan_kernel<M>    each block orders its item's LLMs and, where the item's option table
//                            fits in LDS, builds it there: per (position in the order, first-unit
//                            offset mod Q, fraction) the smallest Eq. 1 contribution among the
//                            options whose units are that fraction and whose replicas fit at that
//                            offset (lowest option among equal ones).  With the fraction vector
//                            fixed the LLMs are independent and L_w is a sum, so this table
//                            decides every vector.  A wave takes prefixes (the first fraction with
//                            3 LLMs, the first two beyond), walks the middle fractions together
//                            and spreads the last free fraction over its lanes; the
//                            lexicographic (L_w, x) minimum and the vector count are reduced per
//                            block, and the item's last block writes the result.
//   pruned_clear_kernel, pruned_scatter_kernel
//                            a table too large for LDS, built in device memory first.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alp_device.h"
#include "alp_internal.h"

namespace alp {

namespace {

// Does an LLM whose units start at offset r (mod Q) and span f units fit d replicas of tp ranks
// of q units, the ranks of a replica on distinct GPUs?  A GPU holding h of its units takes at
// most min(floor(h / q), d) ranks, and the sum reaching tp * d suffices (deal the ranks to the
// replicas GPU by GPU in turn).  The units occupy a partial first GPU, full GPUs, and a partial
// last GPU.  f > 0.  mul_Q divides by Q; inv_q = ceil(2^16 / q) divides h <= Q <= 16: the excess
// h (q - 1) / (q 2^16) stays below 1 / q.
__device__ __forceinline__ bool placement_fits(uint32_t Q, uint32_t mul_Q, uint32_t r, uint32_t f,
                                               uint32_t tp, uint32_t inv_q, uint32_t d)
{
    const uint32_t end = r + f;
    auto take = [&](uint32_t h) { const uint32_t c = (h * inv_q) >> 16; return c < d ? c : d; };
    const uint32_t gpus = div_by(end, mul_Q), tail = end - gpus * Q;
    const uint32_t ranks =
        end <= Q ? take(f) : take(Q - r) + (gpus - 1) * take(Q) + take(tail);
    return ranks >= tp * d;
}

// Table entries pack (c << 32 | option): the 64-bit minimum is the smallest contribution, then
// the lowest option.  No admissible option: all ones (c = kNoLatency).
constexpr uint64_t kNoEntry = ~0ull;

// Largest table staged in LDS (with the static LDS, within the 64 KiB a block gets without an
// opt-in).
constexpr uint64_t kStageBytes = 60 * 1024;
constexpr uint32_t kScanThreads = 512;

// The fractions position k of the order can take: all up to F, or with the ordering flag at most
// F / (k + 1), since no earlier position has fewer.  (k + 1 <= 8: a reciprocal multiplication.)
__host__ __device__ inline uint32_t table_width(uint32_t F, uint32_t k, bool ordered)
{
    return (ordered ? F / (k + 1) : F) + 1;
}

// Entries of the table in LDS for F units: position 0 starts at offset 0 only.
inline uint64_t staged_entries(uint32_t M, uint32_t Q, uint32_t F, bool ordered)
{
    uint64_t n = 0;
    for (uint32_t k = 0; k < M; ++k)
        n += (uint64_t)(k == 0 ? 1 : Q) * table_width(F, k, ordered);
    return n;
}

// Per-item constants of step 1, by position in the latency-ratio order.
struct Order {
    uint32_t lo[ALP_MAX_LLMS], hi[ALP_MAX_LLMS], lo_after[ALP_MAX_LLMS];
    uint32_t llm[ALP_MAX_LLMS];
    uint32_t tab[ALP_MAX_LLMS], width[ALP_MAX_LLMS];   // its table rows: first entry, row length
    uint64_t pw[ALP_MAX_LLMS];      // O^(M-1-m) of the LLM m at the position
    uint32_t empty;
};

__global__ void __launch_bounds__(256)
pruned_clear_kernel(uint64_t entries, uint64_t *__restrict__ table)
{
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < entries)
        table[t] = kNoEntry;
}

// One thread per (item, LLM, option): an option usable at the query (ok and within
// saturation) with u units is admissible for fraction f = u at every first-unit offset r
// (mod Q) where its replicas fit; it enters those entries by a 64-bit minimum.
__global__ void __launch_bounds__(256)
pruned_scatter_kernel(SpaceDev sp, const uint2 *__restrict__ rec, uint32_t count, uint32_t F1,
                      uint32_t mul_Q, uint64_t *__restrict__ table)
{
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (uint64_t)count * sp.M * sp.O)
        return;
    const uint32_t o = (uint32_t)(t % sp.O);
    const uint64_t im = t / sp.O;                       // item * M + m
    const uint2 e = rec[t];
    const uint32_t u = e.y;                             // unusable options carry the sentinel
    if (u >= F1)
        return;
    const uint32_t ij = o / sp.D;
    const uint32_t tp = sp.tp(ij / sp.n_fq), q = sp.fq(ij % sp.n_fq), d = o % sp.D + 1;
    const uint64_t key = ((uint64_t)e.x << 32) | o;
    const uint32_t inv_q = (0xFFFFu + q) / q;
    for (uint32_t r = 0; r < sp.Q; ++r)
        if (placement_fits(sp.Q, mul_Q, r, u, tp, inv_q, d))
            atomicMin((unsigned long long *)&table[(im * sp.Q + r) * F1 + u],
                      (unsigned long long)key);
}

// Fractions fixed per prefix.
template <int M>
constexpr int kPrefix = M <= 2 ? 0 : M == 3 ? 1 : 2;

struct Walk {
    const uint64_t *table;
    uint32_t Q, mul_Q;
    bool ordered, staged;
    uint32_t L;                     // running best (L, x) and vector count of the lane
    uint64_t x;
    uint64_t count;
    __device__ __forceinline__ uint32_t mod_q(uint32_t v) const
    {
        return v - div_by(v, mul_Q) * Q;
    }
};

// Position k receives v units, its first unit at offset r (mod Q): adds the table entry's
// contribution and option (no admissible option: dead).
__device__ __forceinline__ void take(const Order &od, const Walk &w, int k, uint32_t r, uint32_t v,
                                     uint32_t &L, uint64_t &x, bool &alive)
{
    const uint64_t e = w.table[od.tab[k] + r * od.width[k] + v];
    alive = alive && e != kNoEntry;
    L += (uint32_t)(e >> 32);
    x += (uint64_t)(uint32_t)e * od.pw[k];
}

// The range [lo, hi] of position K's fraction given what remains and the fraction before it.
template <int K>
__device__ __forceinline__ void range(const Order &od, const Walk &w, uint32_t remaining,
                                      uint32_t prev, uint32_t &lo, uint32_t &hi)
{
    lo = od.lo[K];
    hi = od.hi[K];
    if (w.ordered && K > 0 && prev < hi)
        hi = prev;
    const bool any = remaining >= od.lo_after[K];
    const uint32_t left = any ? remaining - od.lo_after[K] : 0u;
    hi = left < hi ? left : hi;
    lo = any ? lo : hi + 1;
}

__device__ __forceinline__ uint32_t uniform(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// The free fraction K = M - 2 spread over GROUP lanes (`first` the lane's among them); the last
// one is what remains.
template <int M, int GROUP>
__device__ __forceinline__ void walk_lanes(const Order &od, Walk &w, uint32_t first,
                                           uint32_t offset, uint32_t remaining, uint32_t prev,
                                           uint32_t L, uint64_t x, bool alive)
{
    constexpr int K = M - 2;
    uint32_t lo, hi;
    range<K>(od, w, remaining, prev, lo, hi);
    // The last position's own bounds, as bounds on v: lo <= remaining - v <= min(hi, v).
    const uint32_t last_lo = od.lo[M - 1], last_hi = od.hi[M - 1];
    if (remaining < last_lo)
        return;
    hi = remaining - last_lo < hi ? remaining - last_lo : hi;
    if (remaining > last_hi && remaining - last_hi > lo)
        lo = remaining - last_hi;
    if (w.ordered && (remaining + 1) / 2 > lo)
        lo = (remaining + 1) / 2;
    // A prefix without an allocation is only counted, and a lane without one for K reads no further
    // where that is a read of memory (LDS answers sooner than a branch pays).  4 LLMs, 512 units,
    // 64 queries, tables in device memory: 6,190 us with every read made, 1,277 so; one query of 5
    // LLMs and 160 units, in LDS: 152 and 65.
    if (!alive) {
        if (lo + first <= hi)
            w.count += (hi - lo - first) / GROUP + 1;
        return;
    }
    const uint32_t r0 = w.mod_q(offset);
    for (uint32_t v = lo + first; v <= hi; v += GROUP) {
        uint32_t L2 = L;
        uint64_t x2 = x;
        bool a = true;
        take(od, w, K, r0, v, L2, x2, a);
        if (a || w.staged)
            take(od, w, M - 1, w.mod_q(offset + v), remaining - v, L2, x2, a);
        w.count += 1;
        if (a && lex_less(L2, x2, w.L, w.x)) {
            w.L = L2;
            w.x = x2;
        }
    }
}

// The fractions from position K on.  From 5 LLMs the last middle fraction (M - 3) goes to four
// groups of 16 lanes and the free one to the lanes of a group: with the ordering its range is
// often below 64.
template <int M, int K>
__device__ __forceinline__ void walk_from(const Order &od, Walk &w, uint32_t offset,
                                          uint32_t remaining, uint32_t prev, uint32_t L,
                                          uint64_t x, bool alive)
{
    const uint32_t lane = threadIdx.x & 63;
    if constexpr (K == M - 2) {
        walk_lanes<M, 64>(od, w, lane, offset, remaining, prev, L, x, alive);
    } else {
        constexpr bool split = K == M - 3;
        uint32_t lo, hi;
        range<K>(od, w, remaining, prev, lo, hi);
        if constexpr (split) {
            // the largest of the last three fractions
            if (w.ordered && (remaining + 2) / 3 > lo)
                lo = (remaining + 2) / 3;
            lo += lane >> 4;
        } else {
            lo = uniform(lo);
            hi = uniform(hi);
        }
        const uint32_t r = w.mod_q(offset);
        for (uint32_t v = lo; v <= hi; v += split ? 4 : 1) {
            uint32_t L2 = L;
            uint64_t x2 = x;
            bool a = alive;
            take(od, w, K, r, v, L2, x2, a);
            if constexpr (split)
                walk_lanes<M, 16>(od, w, lane & 15, offset + v, remaining - v, v, L2, x2, a);
            else
                walk_from<M, K + 1>(od, w, offset + v, remaining - v, v, L2, x2, a);
        }
    }
}

// C(F + K, K), saturating at 2^64 - 1: the product of (F + i) / i, i = 1 .. K, exact at every step
// and ascending, in 32-bit digits (F + i < 2^12, divisors known at compile time).
template <int K>
__device__ __forceinline__ uint64_t binomial_sat(uint32_t F)
{
    uint64_t c = 1;
    bool over = false;
#pragma unroll
    for (uint32_t i = 1; i <= (uint32_t)K; ++i) {
        const uint64_t p0 = (c & 0xFFFFFFFFu) * (F + i);
        const uint64_t p1 = (c >> 32) * (F + i) + (p0 >> 32);      // below 2^45
        const uint64_t h = p1 / i;
        const uint64_t l = (((p1 - h * i) << 32) | (p0 & 0xFFFFFFFFu)) / i;
        over = over || (h >> 32) != 0;
        c = (h << 32) + l;
    }
    return over ? ~0ull : c;
}

// The item's order and bounds (step 1), by the first wave: lane m holds LLM m.
__device__ __forceinline__ void item_order(const SpaceDev &sp, const TablesDev &tb, uint32_t inst,
                                           uint32_t F, uint32_t flags, bool staged, uint32_t F1,
                                           Order *od)
{
    const uint32_t lane = threadIdx.x, M = sp.M;
    const bool ordered = (flags & ALP_PRUNE_ORDER) != 0;
    // Latency ratio: the contribution at tp[0], the largest share and the first profiled point,
    // largest first, ties by LLM index.
    uint64_t ref = 0;
    uint32_t need = 0;
    if (lane < M) {
        const uint64_t base = (uint64_t)inst * M + lane;
        const uint64_t cell = (base * sp.n_tp + 0) * sp.n_fq + (sp.n_fq - 1);
        const uint32_t lat = tb.lat[cell * sp.K], n = tb.n[base], p = tb.p[base];
        const uint64_t W = tb.W[base];
        ref = (uint64_t)lat * n / p;
        if (flags & ALP_PRUNE_MIN_FRACTION) {
            const uint64_t u = (W * sp.Q + tb.H - 1) / tb.H;   // above F: more than fits anyway
            need = u > 1 ? (u < 0x10000u ? (uint32_t)u : 0x10000u) : 1u;
        }
    }
    uint32_t pos = 0;
    for (uint32_t m = 0; m < M; ++m) {
        const uint64_t o = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(ref >> 32), (int)m) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ref, (int)m);
        pos += o > ref || (o == ref && m < lane) ? 1u : 0u;
    }
    if (lane < M) {
        od->llm[pos] = lane;
        od->lo[pos] = need;
        uint64_t pw = 1;
        for (uint32_t j = lane + 1; j < M; ++j)
            pw *= sp.O;
        od->pw[pos] = pw;
    }
    // (one wave: its LDS writes are in order with its reads)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) {
        uint64_t after = 0;
        od->empty = 0;
        for (int k = (int)M - 1; k >= 0; --k) {
            uint32_t lo = od->lo[k];
            if (after + lo > F) {
                od->empty = 1;
                lo = 0;
            }
            od->lo[k] = lo;
            od->lo_after[k] = (uint32_t)after;
            od->hi[k] = F - (uint32_t)after;
            after += lo;
        }
        uint32_t at = 0;
        for (uint32_t k = 0; k < M; ++k) {
            const uint32_t width = staged ? table_width(F, k, ordered) : F1;
            od->tab[k] = staged ? at : od->llm[k] * sp.Q * F1;
            od->width[k] = width;
            at += (k == 0 ? 1 : sp.Q) * width;
        }
    }
}

// What bounds it: latency.  The paper's scheduler point (5 LLMs, 16 GPUs, 10 fractions) has
// 241,860 vectors, under 10 us of instructions on the chip, but a thread per prefix walked up to
// 800 of them in turn over a table in device memory (150 us).  A wave per prefix, lanes over the
// last free fraction and the table in LDS (its rows cut to what each position can take: 18 KB
// instead of 64) leave a wave some 50 steps of one LDS round trip.
template <int M>
__global__ void __launch_bounds__(kScanThreads)
pruned_scan_kernel(SpaceDev sp, TablesDev tb, QueryDev q, const uint2 *__restrict__ rec,
                   uint32_t F1, uint32_t mul_Q, uint32_t flags,
                   const uint64_t *__restrict__ table, uint32_t stage, uint32_t blocks_per_item,
                   unsigned long long *__restrict__ slots, uint32_t *__restrict__ counters,
                   const uint2 *__restrict__ ext, alp_pruned_t *__restrict__ out)
{
    extern __shared__ __align__(8) unsigned char s_dyn[];
    __shared__ Order od;
    const uint32_t item = blockIdx.x / blocks_per_item;
    const uint32_t sub = blockIdx.x - item * blocks_per_item;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = blockDim.x >> 6;
    const bool ordered = (flags & ALP_PRUNE_ORDER) != 0;
    uint32_t inst, F, lambda;
    load_query(q, item, inst, F, lambda);
    uint64_t *s_tab = reinterpret_cast<uint64_t *>(s_dyn);
    if (wave == 0)
        item_order(sp, tb, inst, F, flags, stage != 0, F1, &od);
    if (stage) {
        for (uint32_t k = threadIdx.x; k < stage; k += blockDim.x)
            s_tab[k] = kNoEntry;
        __syncthreads();
        // Every usable option enters its fraction's entry at each offset where its replicas fit,
        // by a 64-bit minimum of (c << 32 | option).
        const uint2 *R = rec + (uint64_t)item * M * sp.O;
        for (uint32_t a = threadIdx.x; a < M * sp.O; a += blockDim.x) {
            const uint32_t k = div_by(a, sp.mul_O), o = a - k * sp.O;
            const uint2 e = R[od.llm[k] * sp.O + o];
            if (e.y >= od.width[k])                 // unusable (the sentinel), or too many units
                continue;
            const uint32_t ij = div_by(o, sp.mul_D), i = ij / sp.n_fq;
            const uint32_t tp = sp.tp(i), fq = sp.fq(ij - i * sp.n_fq), d = o - ij * sp.D + 1;
            const unsigned long long key = ((unsigned long long)e.x << 32) | o;
            const uint32_t offsets = k == 0 ? 1u : sp.Q, inv_q = (0xFFFFu + fq) / fq;
            for (uint32_t r = 0; r < offsets; ++r)
                if (placement_fits(sp.Q, mul_Q, r, e.y, tp, inv_q, d))
                    atomicMin(reinterpret_cast<unsigned long long *>(
                                  &s_tab[od.tab[k] + r * od.width[k] + e.y]), key);
        }
    }
    __syncthreads();
    Walk w;
    w.table = stage ? s_tab : table + (uint64_t)item * M * sp.Q * F1;
    w.Q = sp.Q;
    w.mul_Q = mul_Q;
    w.ordered = ordered;
    w.staged = stage != 0;
    w.L = kNoLatency;
    w.x = ~0ull;
    w.count = 0;

    if (!od.empty) {
        const uint32_t first = sub * waves + wave, step = blocks_per_item * waves;
        if constexpr (M == 1) {
            if (first == 0 && lane == 0 && F >= od.lo[0]) {
                uint32_t L = 0;
                uint64_t x = 0;
                bool a = true;
                take(od, w, 0, 0, F, L, x, a);
                w.count = 1;
                if (a) {
                    w.L = L;
                    w.x = x;
                }
            }
        } else if constexpr (M == 2) {
            if (first == 0)
                walk_from<M, 0>(od, w, 0, F, 0, 0, 0, true);
        } else if constexpr (kPrefix<M> == 1) {
            uint32_t lo, hi;
            range<0>(od, w, F, 0, lo, hi);
            lo = uniform(lo);
            hi = uniform(hi);
            for (uint32_t f0 = lo + first; f0 <= hi; f0 += step) {
                uint32_t L = 0;
                uint64_t x = 0;
                bool a = true;
                take(od, w, 0, 0, f0, L, x, a);
                walk_from<M, 1>(od, w, f0, F - f0, f0, L, x, a);
            }
        } else {
            // Pairs (f0, f1) of the rectangle that holds every valid one, f0 major; each wave takes
            // every step-th (neighbours, of like work, go to different waves) and skips those that
            // leave no vector.
            uint32_t lo, hi;
            range<0>(od, w, F, 0, lo, hi);
            if (ordered && (F + M - 1) / M > lo)
                lo = (F + M - 1) / M;                  // the largest of M fractions
            lo = uniform(lo);
            hi = uniform(hi);
            const uint32_t lo1 = uniform(od.lo[1]), after1 = uniform(od.lo_after[1]);
            uint32_t top1 = uniform(od.hi[1]);
            top1 = ordered && F / 2 < top1 ? F / 2 : top1;
            const uint32_t n1 = top1 >= lo1 ? top1 - lo1 + 1 : 0u;
            const uint32_t pairs = hi >= lo ? (hi - lo + 1) * n1 : 0u;
            for (uint32_t t = first; t < pairs; t += step) {
                const uint32_t row = t / n1, f0 = lo + row, f1 = lo1 + (t - row * n1);
                const uint32_t rest = F - f0;
                if (rest < after1 || f1 > rest - after1 ||
                    (ordered && (f1 > f0 || (M - 1) * f1 < rest)))
                    continue;
                uint32_t L = 0;
                uint64_t x = 0;
                bool a = true;
                take(od, w, 0, 0, f0, L, x, a);
                take(od, w, 1, w.mod_q(f0), f1, L, x, a);
                walk_from<M, 2>(od, w, f0 + f1, rest - f1, f1, L, x, a);
            }
        }
    }

    // Block totals: the vector count and the (L, x) winner, by the first wave.
    __shared__ uint64_t s_count[kScanThreads / 64];
    uint64_t total = w.count;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        total += __shfl_xor((unsigned long long)total, off, 64);
    if (lane == 0)
        s_count[wave] = total;
    uint32_t L = w.L;
    uint64_t x = w.x;
    block_min(L, x);                                   // (a barrier: the counts are written)
    if (wave != 0)
        return;
    total = 0;
    for (uint32_t k = 0; k < waves; ++k)
        total += s_count[k];
    if (blocks_per_item > 1) {
        // The block's results in its slots by atomic exchanges, then its count; the item's last
        // block reads every slot, by atomics too.
        unsigned long long *mine = slots + 3 * ((uint64_t)item * blocks_per_item + sub);
        if (lane < 3)
            (void)atomicExch(mine + lane, lane == 0 ? (unsigned long long)L
                                        : lane == 1 ? (unsigned long long)x
                                                    : (unsigned long long)total);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        uint32_t last = 0;
        if (lane == 0)
            last = count_block(counters, item, sub, blocks_per_item) ? 1u : 0u;
        if (!__builtin_amdgcn_readfirstlane((int)last))
            return;
        L = kNoLatency;
        x = ~0ull;
        total = 0;
        for (uint32_t k = lane; k < blocks_per_item; k += 64) {
            unsigned long long *slot = slots + 3 * ((uint64_t)item * blocks_per_item + k);
            const uint32_t l = (uint32_t)atomicOr(slot, 0ull);
            const uint64_t xk = atomicOr(slot + 1, 0ull);
            total += atomicOr(slot + 2, 0ull);
            if (lex_less(l, xk, L, x)) {
                L = l;
                x = xk;
            }
        }
        wave_min(L, x);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
            total += __shfl_xor((unsigned long long)total, off, 64);
    }
    uint64_t *dst = reinterpret_cast<uint64_t *>(out + item);
    write_result(sp, ext + (uint64_t)item * M * sp.O, L, x, dst);
    if (threadIdx.x != 0)
        return;
    dst[6] = total;
    dst[7] = binomial_sat<M - 1>(F);
}

}  // namespace

uint64_t pruned_table_entries(const SpaceDev &sp, uint32_t F_max, uint32_t flags)
{
    const uint64_t staged = staged_entries(sp.M, sp.Q, F_max, (flags & ALP_PRUNE_ORDER) != 0);
    return staged * sizeof(uint64_t) <= kStageBytes ? 0 : (uint64_t)sp.M * sp.Q * (F_max + 1);
}

// About two prefixes a wave (with 3 LLMs a prefix is one fraction, beyond two, of which roughly an
// eighth leave any vector), and at most 512 blocks (two to a CU): every block orders the LLMs and
// builds the table in LDS.  With the tables in device memory a batch takes up to 2,048 blocks, 512
// an item: fewer work on more items at once, whose tables the L2s do not hold (4 LLMs, 512 units,
// 64 queries: 1,277 us at 512 blocks, 1,124 at 2,048; 256 units, 600 queries: 3,203 and 2,530).
uint32_t pruned_blocks_per_item(const SpaceDev &sp, uint32_t F_max, uint32_t flags, uint32_t count)
{
    const uint64_t F1 = (uint64_t)F_max + 1;
    const uint64_t prefixes = sp.M <= 2 ? 1 : sp.M == 3 ? F1 : F1 * F1 / 8;
    const uint64_t want = (prefixes / 2 + kScanThreads / 64 - 1) / (kScanThreads / 64);
    const uint64_t most = pruned_table_entries(sp, F_max, flags) ? 2048 : 512;
    const uint64_t share = most / count, room = share < 1 ? 1 : share < 512 ? share : 512;
    const uint64_t n = want < room ? want : room;
    return n < 1 ? 1u : (uint32_t)n;
}

hipError_t launch_pruned(const SpaceDev &sp, const TablesDev &tb, const QueryDev &q, uint32_t count,
                         uint32_t F_max, uint32_t flags, const uint2 *rec, uint64_t *table,
                         uint32_t blocks_per_item, uint64_t *slots, uint32_t *counters,
                         const uint2 *ext, alp_pruned_t *out, hipStream_t st,
                         hipEvent_t table_done)
{
    if (count == 0)
        return hipSuccess;
    const uint32_t F1 = F_max + 1, mul_Q = div_multiplier(sp.Q);
    hipError_t e;
    uint32_t stage = 0;
    const uint64_t entries = pruned_table_entries(sp, F_max, flags) * count;
    if (entries) {
        hipLaunchKernelGGL(pruned_clear_kernel, dim3((uint32_t)((entries + 255) / 256)), dim3(256),
                           0, st, entries, table);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
        const uint64_t options = (uint64_t)count * sp.M * sp.O;
        hipLaunchKernelGGL(pruned_scatter_kernel, dim3((uint32_t)((options + 255) / 256)),
                           dim3(256), 0, st, sp, rec, count, F1, mul_Q, table);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    } else {
        stage = (uint32_t)staged_entries(sp.M, sp.Q, F_max, (flags & ALP_PRUNE_ORDER) != 0);
    }
    if (table_done && (e = hipEventRecord(table_done, st)) != hipSuccess)
        return e;
    // (a launch holds fewer than 2^32 threads)
    uint32_t threads = kScanThreads;
    while (threads > 64 && (uint64_t)count * blocks_per_item * threads >= (UINT64_C(1) << 32))
        threads /= 2;
    const dim3 grid(count * blocks_per_item), block(threads);
    const size_t lds = (size_t)stage * sizeof(uint64_t);
#define ALP_PRUNED_CASE(MM)                                                                        \
    case MM:                                                                                       \
        hipLaunchKernelGGL(pruned_scan_kernel<MM>, grid, block, lds, st, sp, tb, q, rec, F1, mul_Q, \
                           flags, table, stage, blocks_per_item,                                   \
                           reinterpret_cast<unsigned long long *>(slots), counters, ext, out);     \
        break;
    switch (sp.M) {
        ALP_PRUNED_CASE(1)
        ALP_PRUNED_CASE(2)
        ALP_PRUNED_CASE(3)
        ALP_PRUNED_CASE(4)
        ALP_PRUNED_CASE(5)
        ALP_PRUNED_CASE(6)
        ALP_PRUNED_CASE(7)
        ALP_PRUNED_CASE(8)
    default:
        return hipErrorInvalidValue;
    }
#undef ALP_PRUNED_CASE
    return hipGetLastError();
}

}  // namespace alp
