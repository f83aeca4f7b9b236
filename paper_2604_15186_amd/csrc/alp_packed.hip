// gfx950 scan of the candidate space in packed 16-bit arithmetic: every candidate's budget test
// and latency comparison at one and a quarter VALU lane-operations, in one launch.
//
// Roles of the LLMs.  The last LLM is the "inner" one: its options j are walked by the loop, one
// 32-bit record each, read through the scalar cache.  The two LLMs before it are the "lane" LLMs:
// their pairs e = o_{M-3} * O + o_{M-2} (the options of LLM 0 alone with two LLMs) are spread over
// the lanes, 2 R pairs per lane in chunks of 128 R, so that option counts that fill no wavefront
// waste only the end of the last chunk.  The others are the "outer" LLMs: a row q fixes their
// digits.  A tile is one row and one chunk against every record; the candidate index is
// x = (q * E + e) * O + j, so tiles ascend in index order, then lanes' pairs, then records.
//
// One candidate.  With T the share units that row and pair leave to the inner LLM (0 to U, the
// most any option uses, where U means no limit), the record's units u_j and the rank rho_j of its
// latency term among the inner LLM's usable terms (below S), both scaled so that one unit is S:
//     value = max((u_j - T) * S, rho_j)
// is rho_j if the candidate fits the budget and at least S otherwise, and the minimum over j,
// started at S, is the rank of the lowest latency that fits, or S.  A register holds two pairs,
// a record (u_j * S in the low half, rho_j in the high one) is applied to both by operand
// selection: a packed subtraction and a packed maximum per record, and one packed three-operand
// minimum per two records (on half-precision floats: non-negative patterns below the infinity's
// order like integers, and denormals are kept).  The masked 32-bit form (v_cmpx, v_min_u32 and a
// scalar restore of EXEC) takes two operations per candidate, each behind the previous one's
// EXEC: as a bare loop on one chip 14.1 * 10^12 candidates/s at 8 waves per SIMD and 6.9 at one,
// this one (R = 4) 28.3 and 22.1.
//
// At the end of a tile each pair's rank is turned back into the term (a table in LDS), the pair's
// and the row's terms are added, and only if some lane reaches the wave's best does the wave
// reduce: so the wave always holds its lowest (latency, q * E + e) and nothing is scanned again;
// the block's winner finds its record j by one look over the inner LLM's options.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "alp_device.h"
#include "alp_internal.h"

namespace alp {

namespace {

typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Units of an unusable option: above every budget (at most M * U, below this by the plan's test),
// and the sum of two stays within 16 bits.
constexpr uint32_t kUnusable = 0x7FFFu;

// Four records (a..d, packed as above) against one register of pairs: t_k = u_k * S - T,
// max(t_k, rho_k), and the running minimum.  NARROW: signed, values below the half-precision
// infinity's pattern; WIDE: unsigned with saturation, a minimum per record.
#define ALP_SUB_N(T, S, W) "v_pk_sub_i16 %[" T "], %[" S "], %[" W "] op_sel_hi:[0,1]\n\t"
#define ALP_SUB_W(T, S, W) "v_pk_sub_u16 %[" T "], %[" S "], %[" W "] op_sel_hi:[0,1] clamp\n\t"
#define ALP_MAX_N(T, S) "v_pk_max_i16 %[" T "], %[" T "], %[" S "] op_sel:[0,1] op_sel_hi:[1,1]\n\t"
#define ALP_MAX_W(T, S) "v_pk_max_u16 %[" T "], %[" T "], %[" S "] op_sel:[0,1] op_sel_hi:[1,1]\n\t"
#define ALP_MIN_N(T, U) "v_pk_minimum3_f16 %[b], %[b], %[" T "], %[" U "]\n\t"
#define ALP_MIN_W(T, U)                                                                            \
    "v_pk_min_u16 %[b], %[b], %[" T "]\n\t"                                                        \
    "v_pk_min_u16 %[b], %[b], %[" U "]\n\t"
#define ALP_G4(F, A, B, C, D)                                                                      \
    ALP_SUB_##F("t0", A, "w") ALP_SUB_##F("t1", B, "w") ALP_SUB_##F("t2", C, "w")                  \
        ALP_SUB_##F("t3", D, "w") ALP_MAX_##F("t0", A) ALP_MAX_##F("t1", B) ALP_MAX_##F("t2", C)   \
            ALP_MAX_##F("t3", D) ALP_MIN_##F("t0", "t1") ALP_MIN_##F("t2", "t3")
#define ALP_G16(F)                                                                                 \
    ALP_G4(F, "s0", "s1", "s2", "s3") ALP_G4(F, "s4", "s5", "s6", "s7")                            \
        ALP_G4(F, "s8", "s9", "s10", "s11") ALP_G4(F, "s12", "s13", "s14", "s15")
#define ALP_REC16(x)                                                                               \
    [s0] "s"(x[0]), [s1] "s"(x[1]), [s2] "s"(x[2]), [s3] "s"(x[3]), [s4] "s"(x[4]),                \
        [s5] "s"(x[5]), [s6] "s"(x[6]), [s7] "s"(x[7]), [s8] "s"(x[8]), [s9] "s"(x[9]),            \
        [s10] "s"(x[10]), [s11] "s"(x[11]), [s12] "s"(x[12]), [s13] "s"(x[13]),                    \
        [s14] "s"(x[14]), [s15] "s"(x[15])
#define ALP_TEMPS [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)

__device__ __forceinline__ uint64_t uniform64(const void *p)
{
    const uint64_t a = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// 16 records through the scalar cache (the block wrote them: see scalar_load16 of the row scan).
__device__ __forceinline__ u32x16 load16(uint64_t p)
{
    u32x16 x;
    asm volatile("s_load_dwordx16 %[x], %[p], 0x0\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : [x] "=&s"(x)
                 : [p] "s"(p)
                 : "memory");
    return x;
}

// 16 records against one register of pairs.
template <bool WIDE>
__device__ __forceinline__ void fold16(uint32_t &b, uint32_t w, const u32x16 &x)
{
    uint32_t t0, t1, t2, t3;
    if constexpr (WIDE)
        asm(ALP_G16(W) : [b] "+v"(b), ALP_TEMPS : [w] "v"(w), ALP_REC16(x));
    else
        asm(ALP_G16(N) : [b] "+v"(b), ALP_TEMPS : [w] "v"(w), ALP_REC16(x));
}

// The same while the 16 records at p load; the load is complete when the statement ends.
template <bool WIDE>
__device__ __forceinline__ u32x16 fold16_load(uint32_t &b, uint32_t w, const u32x16 &x, uint64_t p)
{
    uint32_t t0, t1, t2, t3;
    u32x16 nx;
    if constexpr (WIDE)
        asm volatile("s_load_dwordx16 %[nx], %[p], 0x0\n\t" ALP_G16(W) "s_waitcnt lgkmcnt(0)"
                     : [nx] "=&s"(nx), [b] "+v"(b), ALP_TEMPS
                     : [p] "s"(p), [w] "v"(w), ALP_REC16(x)
                     : "memory");
    else
        asm volatile("s_load_dwordx16 %[nx], %[p], 0x0\n\t" ALP_G16(N) "s_waitcnt lgkmcnt(0)"
                     : [nx] "=&s"(nx), [b] "+v"(b), ALP_TEMPS
                     : [p] "s"(p), [w] "v"(w), ALP_REC16(x)
                     : "memory");
    return nx;
}

__device__ __forceinline__ uint32_t pack2(uint32_t lo, uint32_t hi) { return lo | (hi << 16); }

// Writes the result of an item whose lowest latency is L at lanes' index X = q * E + e (L =
// kNoLatency: none), by one wave.  Lane m < M - 1 takes LLM m's option, a digit of X; the sums of
// their terms and units give the term the inner LLM's option has and the units left to it, and
// the lowest such option completes the candidate index.
__device__ __forceinline__ void write_packed_result(const PackedPlan &pk, const uint2 *s_cu,
                                                    const uint2 *s_ext, uint32_t cap_units,
                                                    const FinishArgs &fa, bool rejected,
                                                    uint32_t L, uint64_t X, uint32_t item)
{
    const SpaceDev &sp = fa.sp;
    const uint32_t lane = threadIdx.x & 63, M = sp.M, O = sp.O;
    uint32_t o = 0, T = 0, U = 0;
    uint64_t x = 0;
    if (rejected)
        L = kNoLatency;
    if (L != kNoLatency) {
        uint64_t rest = X;
        for (int m = (int)M - 2; m >= 0; --m) {
            uint32_t d;
            if ((rest >> 32) == 0) {
                // floor(rest / O) or one less by the rounded-down reciprocal
                const uint32_t v = (uint32_t)rest;
                uint32_t t = __umulhi(v, pk.inv_O);
                d = v - t * O;
                if (d >= O) {
                    ++t;
                    d -= O;
                }
                rest = t;
            } else {
                const uint64_t t = rest / O;
                d = (uint32_t)(rest - t * O);
                rest = t;
            }
            o = lane == (uint32_t)m ? d : o;
        }
        uint32_t cs = 0, us = 0;
        if (lane < M - 1) {
            const uint2 cu = s_cu[lane * O + o];
            cs = cu.x;
            us = cu.y;
        }
        // Sums over the first 8 lanes (lane ^ 1, lane ^ 2, the half row's mirror).
        cs += dpp_mov<0xB1>(cs, cs);
        us += dpp_mov<0xB1>(us, us);
        cs += dpp_mov<0x4E>(cs, cs);
        us += dpp_mov<0x4E>(us, us);
        cs += dpp_mov<0x141>(cs, cs);
        us += dpp_mov<0x141>(us, us);
        const uint32_t target = L - (uint32_t)__builtin_amdgcn_readfirstlane((int)cs);
        const uint32_t slack = cap_units - (uint32_t)__builtin_amdgcn_readfirstlane((int)us);
        for (uint32_t j0 = 0; j0 < O; j0 += 64) {
            const uint32_t j = j0 + lane;
            const uint2 cu = s_cu[(M - 1) * O + (j < O ? j : O - 1)];
            const uint64_t hit = __ballot(j < O && cu.x == target && cu.y <= slack &&
                                          cu.y != kUnusable);
            if (hit) {
                const uint32_t jf = j0 + (uint32_t)__builtin_ctzll(hit);
                o = lane == M - 1 ? jf : o;
                x = X * O + jf;
                break;
            }
        }
        if (lane < M) {
            const uint2 e = s_ext[lane * O + o];
            T = e.x;
            U = e.y;
        }
    }
    const uint32_t ij = div_by(o, sp.mul_D);
    write_result_lanes(sp, o, ij, div_by(ij, pk.mul_fq), T, U, L, x,
                       reinterpret_cast<uint64_t *>(fa.out + item),
                       rejected ? (uint32_t)ALP_EINVAL : (uint32_t)ALP_INFEASIBLE, fa.signal,
                       fa.seq);
}

template <int R, bool WIDE>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8)))
scan_packed_kernel(QueryDev q, PackedPlan pk, uint32_t blocks_per_item, uint32_t nblocks,
                   FinishArgs fa, FusedArgs fz)
{
    const SpaceDev &sp = fa.sp;
    const uint32_t M = sp.M, O = sp.O;
    // Every line of kernel arguments the prologue reads, in one round trip (see scan_min_kernel).
    asm volatile("" ::"s"(M), "s"(nblocks), "s"(fa.sp.tp8), "s"(fa.out), "s"(fz.tb.rate),
                 "s"(fz.raw.budget), "s"(fz.regions), "s"(fz.slots), "s"(pk.rows),
                 "s"(blockDim.x));
    const uint32_t lb = xcd_logical_block(blockIdx.x, nblocks);
    const uint32_t item = lb / blocks_per_item;
    const uint32_t sub = lb - item * blocks_per_item;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = blockDim.x >> 6;

    // ---- the item's option terms -------------------------------------------------------------
    extern __shared__ uint4 s_dyn[];
    __shared__ LlmInputs s_llm[ALP_MAX_LLMS];
    __shared__ uint32_t s_tpq[ALP_MAX_TP * ALP_MAX_FRAC];
    __shared__ double s_inv_dd[ALP_MAX_REPLICAS];
    __shared__ uint32_t s_wave_L[16];
    __shared__ uint64_t s_wave_E[16];
    __shared__ uint2 s_nothing;
    uint8_t *s_base = reinterpret_cast<uint8_t *>(s_dyn);
    uint32_t *s_rate = reinterpret_cast<uint32_t *>(s_base);
    uint32_t *s_lat = reinterpret_cast<uint32_t *>(s_base + fused_lds_lat_offset(sp));
    uint8_t *s_deploy = s_base + fused_lds_deploy_offset(sp);
    uint32_t *s_key = reinterpret_cast<uint32_t *>(s_base + packed_lds_key_offset(sp));
    uint2 *s_ext = reinterpret_cast<uint2 *>(s_base + packed_lds_ext_offset(sp));
    uint2 *s_cu = s_ext + M * O;              // (c, units), units kUnusable where unusable
    uint32_t *s_term = reinterpret_cast<uint32_t *>(s_cu + M * O);   // rank -> term, S -> none
    const FusedLds flds{s_rate, s_lat, s_deploy, s_tpq, s_llm, s_inv_dd, s_ext};
    uint32_t inst, cap, lambda;
    bool rejected;
    load_item_query(fz.raw, q, item, inst, cap, lambda, rejected);
    stage_item_tables(sp, fz.tb, M, inst, wave, s_rate, s_lat, s_deploy, s_tpq, s_llm, s_inv_dd);
    const uint32_t padded = inner_stride(O);
    for (uint32_t a = threadIdx.x; a < M * O; a += blockDim.x) {
        const uint32_t m = div_by(a, sp.mul_O), o = a - m * O;
        const OptionTerm t = flds.term(sp, m, o, lambda);
        s_ext[a] = make_uint2(t.tau, t.u);
        const bool usable = t.ok && t.thr;
        s_cu[a] = make_uint2(usable ? t.c : 0u, usable ? div_by(t.u, pk.mul_unit) : kUnusable);
        if (m == M - 1)
            s_key[o] = usable ? t.c : kNoLatency;
    }
    for (uint32_t a = O + threadIdx.x; a < padded; a += blockDim.x)
        s_key[a] = kNoLatency;
    if (threadIdx.x == 0) {
        s_term[pk.S] = kNoLatency;
        s_nothing = make_uint2(0u, 0u);
    }
    __syncthreads();
    // The inner LLM's ranks: the number of usable terms below an option's own (equal terms share
    // a rank), counted by four threads per option, and the packed records, written to the block's
    // region and read back through the scalar cache.
    uint32_t *region = reinterpret_cast<uint32_t *>(fz.regions) + (uint64_t)blockIdx.x * padded;
    for (uint32_t i = threadIdx.x; i < 4 * padded; i += blockDim.x) {
        const uint32_t j = i >> 2, part = i & 3;
        const uint32_t mine = s_key[j];
        const uint4 *k4 = reinterpret_cast<const uint4 *>(s_key);
        uint32_t below = 0;
        for (uint32_t k = part; k < padded / 4; k += 4) {
            const uint4 v = k4[k];
            below += (v.x < mine) + (v.y < mine) + (v.z < mine) + (v.w < mine);
        }
        below += dpp_mov<0xB1>(below, below);
        below += dpp_mov<0x4E>(below, below);
        if (part == 0) {
            uint32_t rec = pack2((pk.U + 1) * pk.S, pk.S);
            if (mine != kNoLatency) {
                rec = pack2(s_cu[(M - 1) * O + j].y * pk.S, below);
                s_term[below] = mine;
            }
            region[j] = rec;
        }
    }

    // ---- the block's tiles -------------------------------------------------------------------
    // Tiles are numbered t = q * chunks + chunk, in index order, and a block owns consecutive
    // ones.  With whole rows (rows_per_block > 0) a wave keeps its chunks and walks the block's
    // rows, so that the lanes' set-up is paid once per chunk; otherwise the waves take the block's
    // tiles in turn, which balances any number of them.  Blocks of fewer tiles (or chunks) than
    // waves share each by ranges of the rows or the records.
    uint64_t q0 = 0, q1 = 1;
    uint32_t first, end, j_lo = 0, j_hi = padded;       // the wave's chunks, or the block's tiles
    const bool by_rows = pk.rows_per_block != 0;
    if (by_rows) {
        q0 = (uint64_t)sub * pk.rows_per_block;
        q1 = q0 + pk.rows_per_block < pk.rows ? q0 + pk.rows_per_block : pk.rows;
        first = wave;
        end = pk.chunks;
    } else {
        first = sub * pk.tiles_per_block + wave;
        end = (sub + 1) * pk.tiles_per_block;
        end = end < pk.tiles ? end : pk.tiles;
    }
    const uint32_t n_own = end - (first - wave);
    if (n_own < waves) {
        const uint32_t phases = waves / n_own, phase = wave / n_own;
        first = phase < phases ? first - phase * n_own : end;
        const uint64_t nr = q1 - q0;
        if (by_rows && nr >= phases) {
            q1 = q0 + nr * (phase + 1) / phases;
            q0 = q0 + nr * phase / phases;
        } else {
            j_lo = padded / 16 * phase / phases * 16;
            j_hi = padded / 16 * (phase + 1) / phases * 16;
            first = j_lo < j_hi ? first : end;
        }
    }
    const uint32_t n_outer = M > 3 ? M - 3 : 0;
    // The lane LLMs' and the last outer LLM's options; an LLM that the space lacks is one option
    // of nothing.
    const uint2 *lane_a = M > 2 ? s_cu + (M - 3) * O : &s_nothing, *lane_b = s_cu + (M - 2) * O;
    const uint2 *outer_last = n_outer > 0 ? s_cu + (M - 4) * O : &s_nothing;
    const uint32_t cap_units = [&]() {
        const uint32_t v = div_by(cap, pk.mul_unit);
        return v < M * pk.U ? v : M * pk.U;
    }();
    const u16x2 u2 = {(uint16_t)pk.U, (uint16_t)pk.U};
    const u16x2 s2 = {(uint16_t)pk.S, (uint16_t)pk.S};
    const uint64_t rec_lo = uniform64(region + j_lo), rec_end = rec_lo + 4ull * (j_hi - j_lo);

    // The wave's lowest (latency, q * E + e): the latency of a feasible candidate is below
    // 2^32 - 1, so the start value admits every one of them.
    uint32_t wave_L = kNoLatency - 1;
    uint64_t wave_E = ~0ull;
    if (first >= end)
        __syncthreads();                          // the other waves' records
    else {
        u32x16 x;
        for (uint32_t t = first; t < end; t += waves) {
            uint32_t chunk = t;
            if (!by_rows) {
                const uint32_t row = t / pk.chunks;
                chunk = t - row * pk.chunks;
                q0 = row;
                q1 = q0 + 1;
            }
            // The lanes' pairs: every read at an index clamped into the tables, all in flight
            // together.  Options filling whole waves (O a multiple of 64) give 64 consecutive
            // pairs one first option, found by scalar arithmetic.
            const uint32_t base = chunk * (128u * R), e0 = base + lane;
            uint32_t c_e[2 * R], a_e[R];
            {
                uint2 va[2 * R], vb[2 * R];
                if (O % 64 == 0) {
#pragma unroll
                    for (int k = 0; k < 2 * R; ++k) {
                        const uint32_t eb = base + 64u * k < pk.E ? base + 64u * k : pk.E - 64;
                        const uint32_t p = __umulhi(eb, sp.mul_O);
                        vb[k] = lane_b[eb - p * O + lane];
                        va[k] = lane_a[p];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 2 * R; ++k) {
                        const uint32_t e = e0 + 64u * k < pk.E ? e0 + 64u * k : pk.E - 1;
                        const uint32_t p = __umulhi(e, sp.mul_O);
                        vb[k] = lane_b[e - p * O];
                        va[k] = lane_a[p];
                    }
                }
#pragma unroll
                for (int k = 0; k < 2 * R; ++k)
                    c_e[k] = va[k].x + vb[k].x;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t lo = va[2 * r].y + vb[2 * r].y;
                    const uint32_t hi = va[2 * r + 1].y + vb[2 * r + 1].y;
                    a_e[r] = pack2(e0 + 128u * r < pk.E ? lo : 0xFFFFu,
                                   e0 + 128u * r + 64u < pk.E ? hi : 0xFFFFu);
                }
            }
            if (t == first) {
                // The records have reached L2 (each wave waits for its own stores, which its
                // lanes' set-up has covered) before any wave reads them.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                x = load16(rec_lo);
            }
            // Rows in runs over which only the last outer digit moves; the other digits' sums are
            // taken once per run.
            uint64_t row = q0;
            uint32_t digit = 0, run = 0, oc0 = 0, ou0 = 0;
            for (; row < q1; ++row, ++digit, --run) {
                if (run == 0) {
                    run = 1;
                    if (n_outer > 0) {
                        uint64_t hi = (row >> 32) == 0 ? (uint32_t)row / O : row / O;
                        digit = (uint32_t)(row - hi * O);
                        run = O - digit;
                        oc0 = ou0 = 0;
#pragma unroll 1
                        for (int k = (int)n_outer - 2; k >= 0; --k) {
                            const uint64_t h2 = (hi >> 32) == 0 ? (uint32_t)hi / O : hi / O;
                            const uint2 v = s_cu[(uint32_t)k * O + (uint32_t)(hi - h2 * O)];
                            hi = h2;
                            oc0 += (uint32_t)__builtin_amdgcn_readfirstlane((int)v.x);
                            ou0 += (uint32_t)__builtin_amdgcn_readfirstlane((int)v.y);
                        }
                    }
                }
                const uint2 vo = outer_last[digit];
                const uint32_t oc = oc0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)vo.x);
                const uint32_t ou = ou0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)vo.y);
                // Units the row leaves to the other three LLMs, at most what they can use.
                uint32_t left = cap_units > ou ? cap_units - ou : 0u;
                left = left < 3 * pk.U ? left : 3 * pk.U;
                const u16x2 left2 = {(uint16_t)left, (uint16_t)left};
                uint32_t w[R], b[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    u16x2 t = __builtin_bit_cast(u16x2, a_e[r]);
                    t = __builtin_elementwise_min(__builtin_elementwise_sub_sat(left2, t), u2) * s2;
                    w[r] = __builtin_bit_cast(uint32_t, t);
                    b[r] = pack2(pk.S, pk.S);
                }
                for (uint64_t p = rec_lo; p != rec_end;) {
                    const uint64_t pn = p + 64 == rec_end ? rec_lo : p + 64;
                    const u32x16 nx = fold16_load<WIDE>(b[0], w[0], x, pn);
#pragma unroll
                    for (int r = 1; r < R; ++r)
                        fold16<WIDE>(b[r], w[r], x);
                    x = nx;
                    p += 64;
                }
                // The pairs' lowest latencies (no feasible record: rank S, saturating).
                uint32_t v[2 * R];
                uint32_t low = kNoLatency;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    v[2 * r] = s_term[b[r] & 0xFFFFu];
                    v[2 * r + 1] = s_term[b[r] >> 16];
                }
#pragma unroll
                for (int k = 0; k < 2 * R; ++k) {
                    v[k] = __builtin_elementwise_add_sat(v[k], c_e[k]);
                    low = v[k] < low ? v[k] : low;
                }
                low = __builtin_elementwise_add_sat(low, oc);
                if (__ballot(low <= wave_L)) {
                    const uint32_t L = wave_min_u32(low);
                    uint32_t e = 0xFFFFFFFFu;
#pragma unroll
                    for (int k = 2 * R - 1; k >= 0; --k)
                        e = __builtin_elementwise_add_sat(v[k], oc) == L ? e0 + 64u * k : e;
                    const uint64_t qe = row * pk.E + wave_min_u32(e);
                    if (L < wave_L || qe < wave_E) {
                        wave_L = L;
                        wave_E = qe;
                    }
                }
            }
        }
    }
    // End of the block, by its first wave alone: the lowest (latency, q * E + e) over the waves.
    if (wave_E == ~0ull)
        wave_L = kNoLatency;
    if (lane == 0) {
        s_wave_L[wave] = wave_L;
        s_wave_E[wave] = wave_E;
    }
    __syncthreads();
    if (wave != 0)
        return;
    uint32_t L = lane < waves ? s_wave_L[lane] : kNoLatency;
    uint64_t X = lane < waves ? s_wave_E[lane] : ~0ull;
    if (pk.wide_index) {
        wave_min(L, X);
    } else {
        const uint64_t k = wave_min_u64(((uint64_t)L << 32) | (uint32_t)X);
        L = (uint32_t)(k >> 32);
        X = (uint32_t)k;
    }
    if (blocks_per_item > 1) {
        // Equal tiles end together, so nothing may queue behind the item's other blocks: each
        // block puts its winner in its own slot (one word, (L, X), unless X needs more; atomic
        // exchanges, performed at the agent's point of coherence once they return) and counts
        // itself; the item's last block reads every slot, by atomics too.  (One word raised by
        // atomic maxima, with groups of 64 in one line, cost the 4-LLM search of 256 blocks 8 us.)
        unsigned long long *slots =
            fz.slots + (uint64_t)item * blocks_per_item * (pk.wide_index ? 2 : 1);
        uint32_t last = 0;
        if (lane == 0) {
            if (pk.wide_index) {
                (void)atomicExch(slots + 2 * (uint64_t)sub, (unsigned long long)L);
                (void)atomicExch(slots + 2 * (uint64_t)sub + 1, (unsigned long long)X);
            } else {
                (void)atomicExch(slots + sub, ((unsigned long long)L << 32) | (uint32_t)X);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            last = count_block(fz.group_done, item, sub, blocks_per_item) ? 1u : 0u;
        }
        if (!__builtin_amdgcn_readfirstlane((int)last))
            return;
        L = kNoLatency;
        X = ~0ull;
        if (pk.wide_index) {
            for (uint32_t k = lane; k < blocks_per_item; k += 64) {
                const uint32_t l = (uint32_t)atomicOr(slots + 2 * (uint64_t)k, 0ull);
                const uint64_t x = atomicOr(slots + 2 * (uint64_t)k + 1, 0ull);
                if (lex_less(l, x, L, X)) {
                    L = l;
                    X = x;
                }
            }
            wave_min(L, X);
        } else {
            uint64_t low = ~0ull;
            for (uint32_t k0 = lane; k0 < blocks_per_item; k0 += 8 * 64) {
                uint64_t v[8];
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    v[t] = k0 + 64u * t < blocks_per_item ? atomicOr(slots + k0 + 64u * t, 0ull)
                                                          : ~0ull;
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    low = v[t] < low ? v[t] : low;
            }
            low = wave_min_u64(low);
            L = (uint32_t)(low >> 32);
            X = (uint32_t)low;
        }
    }
    write_packed_result(pk, s_cu, s_ext, cap_units, fa, rejected, L, X, item);
}

}  // namespace

hipError_t launch_packed(const SpaceDev &sp, const QueryDev &q, uint32_t count,
                         const ScanGeometry &g, const FinishArgs &fa, const FusedArgs &fz,
                         hipStream_t st, hipEvent_t t0, hipEvent_t t1)
{
    if (count == 0)
        return hipSuccess;
    const uint32_t nblocks = count * g.blocks_per_item;
    const size_t lds = packed_lds_bytes(sp, g.packed.S);
#define ALP_LAUNCH_PACKED(RR, WW)                                                                  \
    hipExtLaunchKernelGGL(HIP_KERNEL_NAME(scan_packed_kernel<RR, WW>), dim3(nblocks),              \
                          dim3(g.threads), lds, st, t0, t1, 0, q, g.packed, g.blocks_per_item,     \
                          nblocks, fa, fz)
    if (g.packed.wide) {
        switch (g.slots) {
        case 1: ALP_LAUNCH_PACKED(1, true); break;
        case 2: ALP_LAUNCH_PACKED(2, true); break;
        case 4: ALP_LAUNCH_PACKED(4, true); break;
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (g.slots) {
        case 1: ALP_LAUNCH_PACKED(1, false); break;
        case 2: ALP_LAUNCH_PACKED(2, false); break;
        case 4: ALP_LAUNCH_PACKED(4, false); break;
        default: return hipErrorInvalidValue;
        }
    }
#undef ALP_LAUNCH_PACKED
    return hipGetLastError();
}

}  // namespace alp
