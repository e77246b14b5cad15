// Decode attention, matrix-core family, for several query heads per kv-head: every operand of the
// matrix instructions is made in registers, tile by tile, and the packed data arrives in LDS by
// asynchronous copies.
//
// decode_mfma_kernel (kivi_decode_mfma.hip) stages the small operands -- q_c s_c for the keys,
// p_t s_t,g for the values, both as fp16 hi + lo parts in two matrix columns -- through LDS: a
// lane computes a few products per head, writes them, and reads its operand fragment back.  That is
// about 35 vector instructions and eight LDS instructions per head and tile in one dependent chain.
// Here lane (n = lane % 16, kb = lane / 16) computes exactly the eight contraction elements that it
// has to hand to the instruction as column n, for its own head, so all heads of a tile cost the same
// instructions as one and nothing goes through LDS:
//   column n -> head n % HP, hi part (n < 8) or lo part (n >= 8); with HP < 8 the spare column
//   bits select among the channel groups (below).
//   keys  : x = q' s by packed fp16 arithmetic.  operand = RN(q' s - t) with t = 0 in the hi columns (operand = RN(q' s)) and
//           t = RN(q' s) in the lo columns (operand = the remainder,
//           which is exact unless it leaves fp16's range).  q' is the query times a power of two
//           that puts its largest element into [2^8, 2^9): with s < 64 nothing overflows and the
//           remainder keeps 2^-33 of the largest product.  In a tile with a larger scale (wave-uniform
//           branch) the heads whose products would overflow take s 2^-9.
//   logits: a column pair's hi and lo sums meet by one rotation inside the 16 lanes of a row;
//           every lane then has eight logits of its head.  Softmax against a running maximum with
//           4 bits of slack: the state is rescaled only when a logit passes the reference by 2^4.
//   values: the probabilities, split into fp16 hi + lo, change place between the halves of the
//           wavefront by v_permlane32_swap; the order in which a lane reads the key tile's rows is chosen
//           so that this puts tokens 8 kb .. 8 kb + 7 into lane kb, which is the value tile's order.
//           operand = (p_hi + p_lo) s, again as RN and exact remainder.  There are four channel groups,
//           i.e. four operands per tile with HP = 8; with HP = 4 the columns of a head hold two groups
//           at once and with HP = 2 all four, so that the tile takes two operands or one (a matrix
//           instruction of group g fills the columns of the other groups with sums that nobody reads).
//   zero-points: keys by a 16x16x128 product (all rows alike, so every lane gets its head's sum), or, with HP < 8, by dot products of eight
//           channels in each of the four columns that share a head and kb, and six exchanges: 12 vector instructions in place of four
//           of the matrix unit's, which take as long as 25 (the two units hardly overlap: 16 matrix instructions and 64 others of
//           three wavefronts take nine tenths of the sum of their times).  Values by one product with the rows = channel groups.
//   Both exponents hold for ordinary data at no cost per tile.  Larger key scales and value scales are looked at
//   together with what they meet -- the query's channel, the probabilities -- and scaled down only if the products need
//   it; the value exponent falls back when large scales are past.  (Error against 64 bits with a key channel 2^15
//   times larger than the others, or values of 40 000 among values of 1/16: 1e-6 to 5e-6 of the output.)
// Counted over whole launches (2 bits, G = 32; rows, merges and all): 323 vector and 17 matrix instructions per tile at HP = 4
// for four heads, 415 and 22 at HP = 8 for eight, 427 and 23 for runs of eight of 71.
//
// Packed data: `global_load_lds` copies a tile (codes, and the four scale / zero-point rows with one
// instruction) straight into the wavefront's own ring of LDS slots, NB tiles ahead, across unit
// borders.  No registers are held by data in flight, no barrier is needed (each wavefront reads
// only its own ring), and the wait is one vmcnt with a constant.  The copies are issued from inline asm
// because the compiler makes every LDS read wait for all such copies in flight when it knows of them; they
// have no output registers, and extra vector-memory operations by the compiler only make the explicit
// waits stricter.
//
// Tiles that hold fp16 rows (and tiles in which K and V are split differently) are served by workgroups
// of their own in the same launch (or one before it), one or more per unit: key rows are matrix operands as they are; value
// rows meet the fp32 probabilities in 16x16x4 fp32 products; packed parts go through a ring slot.  (Inside the pipelined workgroups that path cost 30 us:
// its loads queue behind the copies in flight and its registers do not fit beside the loop's.)
//
// A step in which a tile leaves the window (K and V split alike, G = 32): the last wavefront of a unit's first row workgroup quantises it
// out of the rings into the cache and a ring slot and attends to it there, the others take the rows.  (Of the units that
// share a kv-head only the first stores it.)  Against a launch of its own before the attention (4.5-5 us), whole steps: 32 / 8
// heads, batch 4, 32 767 tokens 35.3 -> 32.2 us; 71 / 1, batch 16, 4095 tokens 33.9 -> 30.3; 16 / 8, 32 / 8, 64 / 8 heads, batch 4, 2047
// tokens 15.7 -> 13.6, 18.7 -> 15.9, 19.2 -> 16.5, 4 bits 16.0 -> 14.3, 15.8 -> 14.7, 19.2 -> 17.4.
//
// Work: every (batch, kv-head, run of query heads) unit has its steps (4 tiles, one per wavefront of a
// workgroup) on an axis that is cut into one interval per resident workgroup (kivi_tiles_plan.h); a workgroup that
// owns part of a unit leaves a part (m, l, o[128]) per head in the workspace, the last one merges.
//
// Bound: issue (three wavefronts per SIMD; a tile costs its SIMD ~1060 cycles at HP = 4, 1190 at HP = 8: 2.6 for a vector
// instruction, 16 for a matrix one, hardly overlapped; waits for data are 2 %; the copies alone would stream twice as fast),
// and what each launch pays once: 4.4-5 us until the first tile is done with, 1.3-2.1 us to leave a unit, 1 us to be counted,
// 2.2-3.5 us for the merge.
// Whole steps at 2 bits, decode_mfma_kernel / this kernel at first / now: 32 / 8 heads, batch 4, 32 767 tokens 47.2 / 32.1 / 30.4 us
// (3.4 TB/s); 64 / 8 heads, batch 4, 16 377 tokens 48.4 / 30.2 / 25.9; 71 / 1 heads, batch 16, 4095 tokens 70.6 / 30.4 / 25.4.  Error against 64 bits 5e-6 to 1e-5 of the
// output (there 1e-4: codes are placed high in the mantissa here, and the matrix unit aligns products by their nominal
// exponent).
#include "kivi_internal.h"
#include "kivi_quantize_tile.h"
#include "kivi_tiles_plan.h"

#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace kivi {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

union Frag {            // one lane's share of a 16x16x32 fp16 operand: eight halves
    half8 h;
    half2v p[4];
    uint32_t r[4];
};

constexpr float kKeyUnscale = 4194304.0f;      // 2^22: key codes enter as code * 4^r * 2^-22
constexpr float kValueUnscale = 262144.0f;     // 2^18: value codes enter as code * 2^-18 (times 4 in registers 1 and 3 at 2 bits)
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kSlack = 4;                      // log2 headroom of the running softmax reference
constexpr int kQueryExp = 8;                   // largest |q'| lies in [2^8, 2^9)
constexpr uint32_t kKeyScaleLimit = 0x54005400u;       // two times fp16 64.0
constexpr int kKeyScaleShift = 9;              // a head for which such a tile has products above kProductLimit takes s 2^-9
constexpr uint32_t kProductLimit = 0x78007800u;        // two times fp16 2^15
// Value side: p' = p 2^kProbExp, value scales taken as s 2^-ks with s 2^-ks < 2^kValueTop, so that
// p' s < 2^16 with the slack.  4-bit codes: scales are 5 times smaller for the same data.  Scales down to 2^-kValueWindow of
// that need no shift.  Larger ones are taken as they are too while their products stay below 2^11 (kValueProductLimit).
template <int BITS> constexpr int kProbExp = BITS == 2 ? 8 : 11;
template <int BITS> constexpr int kValueTop = BITS == 2 ? 3 : 0;
constexpr int kValueWindow = 7;
constexpr float kValueProductLimit = 2048.f;

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
constexpr int kDppRor8 = 0x128;                // rotate by 8 within 16: the hi and lo column of a head
constexpr int kHiLanes = 0x3, kLoLanes = 0xC;  // bank masks: columns 0-7, columns 8-15
constexpr int kDppRor4 = 0x124;
// sum over the lanes that differ in bits 4 and 5
__device__ __forceinline__ float add_rows(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    x = __int_as_float(a[0]) + __int_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
    return __int_as_float(b[0]) + __int_as_float(b[1]);
}
__device__ __forceinline__ float max_rows(float x) {
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    x = fmaxf(__int_as_float(a[0]), __int_as_float(a[1]));
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
    return fmaxf(__int_as_float(b[0]), __int_as_float(b[1]));
}
// over the 16 lanes of a row
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141;
__device__ __forceinline__ float row_max(float x) {
    x = fmaxf(x, dpp<kDppXor1>(x));
    x = fmaxf(x, dpp<kDppXor2>(x));
    x = fmaxf(x, dpp<kDppHalfMirror>(x));
    return fmaxf(x, dpp<kDppRor8>(x));
}
__device__ __forceinline__ float row_sum(float x) {
    x += dpp<kDppXor1>(x);
    x += dpp<kDppXor2>(x);
    x += dpp<kDppHalfMirror>(x);
    return x + dpp<kDppRor8>(x);
}
// over the 32 lanes of a half of the wavefront
__device__ __forceinline__ float half_max(float x) {
    x = row_max(x);
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    return fmaxf(__int_as_float(a[0]), __int_as_float(a[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    x = row_sum(x);
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    return __int_as_float(a[0]) + __int_as_float(a[1]);
}
// `x` of the partner column in the lanes of BANKS, `own` in the others
template <int BANKS>
__device__ __forceinline__ half2v from_partner(half2v own, half2v x) {
    return __builtin_bit_cast(half2v, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, own), __builtin_bit_cast(int, x), kDppRor8, 0xF, BANKS, false));
}

__device__ __forceinline__ int ring_slot(int start, int i, int cap) {
    int s = start + i;
    s -= (s >= cap) ? cap : 0;
    return s;
}

// Workgroup barrier that orders LDS traffic only (a __syncthreads() would also wait for the copies in flight).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ void wave_lds_sync() {      // LDS instructions of one wavefront execute in order
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// device-scope accesses for the parts (see decode_mfma_kernel: published without cache flushes)
__device__ __forceinline__ void device_store(float* p, float2 v) {
    __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-uniform read of a table that an earlier launch made, through the scalar cache: a vector load would return
// behind all copies in flight.
__device__ __forceinline__ int table(const int32_t* base, int i) {
    return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(base))[i];
}

// Asynchronous copy of 16 bytes per lane: lane l's bytes land at LDS offset lds + 16 l.  (Five wait states between a vector
// instruction that writes the scalar operand, a readlane out of a spill say, and this one: the compiler does not look into the block.  m0 holds the offset; it is a reserved
// register, so the compiler warns that it will not keep a value in it across the statement: nor shall it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_to_lds(const void* base, uint32_t lane_offset, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(lane_offset), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void copy_to_lds(const void* lane_ptr, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds), "v"(lane_ptr) : "memory", "m0");
}
#pragma clang diagnostic pop
// Outputs (two channels at po, two 64 channels further) of the parts first, first + 1, ..., 0 past the last part: all
// device-scope loads are issued before the first is used.  (Two pairs apart and not four channels in a row, so that a
// wavefront's load covers whole memory segments.)  `first` is wave-uniform: what is not there is not loaded.
template <int N>
__device__ __forceinline__ void load_parts(const float* po, int first, int parts, uint64_t (&v)[N][2]) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        v[j][0] = v[j][1] = 0;
        if (first + j < parts) {
            const uint64_t* a = reinterpret_cast<const uint64_t*>(po + (int64_t)(first + j) * kHeadDim);
            v[j][0] = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            v[j][1] = __hip_atomic_load(a + 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}
template <int N>
__device__ __forceinline__ void wait_copies() {        // at most N vector-memory operations still in flight
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ half2v pack_rtz(float a, float b) {
    return __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(a, b));
}
__device__ __forceinline__ half2v half2_of(uint32_t x) { return __builtin_bit_cast(half2v, x); }

// Code fragments of tile coordinate u = 2 pair + odd: a code moved to bit `off` of an fp16 lane is the
// exact subnormal number code * 2^(off - 24).  The instruction aligns products by the operands' nominal
// exponents (2^-14 for every subnormal), so a code near the bottom of the mantissa costs accuracy: the
// shifts put the codes as high as the 10 mantissa bits allow.
//   keys  : bits 2, 4, 6, 8 (2-bit codes), 2, 6 (4-bit): one shift per half-tile; the factors 4^r (16^(r & 1)) are
//           divided out of the query once per unit
//   values: bits 6, 8 (2-bit: factor 4 in registers 1 and 3), 6 (4-bit): more shifts, but p s keeps its range
template <int BITS>
__device__ __forceinline__ half8 key_fragment(const uint32_t* w, int pair, int odd) {
    Frag f;
    if constexpr (BITS == 2) {
        const uint32_t x = odd ? w[pair] >> 6 : w[pair] << 2;
        f.r[0] = x & 0x000C000Cu; f.r[1] = x & 0x00300030u;
        f.r[2] = x & 0x00C000C0u; f.r[3] = x & 0x03000300u;
    } else {
        const uint32_t x0 = odd ? w[pair * 2] >> 6 : w[pair * 2] << 2, x1 = odd ? w[pair * 2 + 1] >> 6 : w[pair * 2 + 1] << 2;
        f.r[0] = x0 & 0x003C003Cu; f.r[1] = x0 & 0x03C003C0u;
        f.r[2] = x1 & 0x003C003Cu; f.r[3] = x1 & 0x03C003C0u;
    }
    return f.h;
}
template <int BITS>
__device__ __forceinline__ half8 value_fragment(const uint32_t* w, int pair, int odd) {
    Frag f;
    if constexpr (BITS == 2) {
        const uint32_t x = odd ? w[pair] >> 2 : w[pair] << 6, y = odd ? w[pair] >> 6 : w[pair] << 2;
        f.r[0] = x & 0x00C000C0u; f.r[1] = x & 0x03000300u;
        f.r[2] = y & 0x00C000C0u; f.r[3] = y & 0x03000300u;
    } else {
        const uint32_t w0 = w[pair * 2], w1 = w[pair * 2 + 1];
        f.r[0] = (odd ? w0 >> 2 : w0 << 6) & 0x03C003C0u; f.r[1] = (odd ? w0 >> 6 : w0 << 2) & 0x03C003C0u;
        f.r[2] = (odd ? w1 >> 2 : w1 << 6) & 0x03C003C0u; f.r[3] = (odd ? w1 >> 6 : w1 << 2) & 0x03C003C0u;
    }
    return f.h;
}

constexpr int kWaves = kStepTiles;             // wavefronts per workgroup
constexpr int kLdsBytes = 160 * 1024 / 3 / 1280 * 1280;    // three workgroups per compute unit (LDS is given out in pieces of 1280 bytes)
// parts of one unit, at most (their statistics meet in LDS)
constexpr int max_parts_of(int bits, int hp) { return bits == 4 && hp == 8 ? kTilesMaxParts / 2 : kTilesMaxParts; }

// The kernel's scalar divisions by numbers that the launch fixes (by_steps: of a unit).  Not in DecodeParams: 56 bytes more cost a
// launch of the other kernels 0.1 us.
struct TilesParams : DecodeParams {
    FastDiv by_runs, by_kv_heads, by_unit_wgs, by_row_split, by_steps, by_axis_longer, by_axis_len;
};

// kWhole: K and V split at the same token, so a tile is all quantised or all fp16; kMixed: any split.
// kQuantisedRagged: the all-quantised tiles of a batch of sequences of different lengths (work cut by tables that
// launch_ragged_rows made or the host did); part 0 of every unit is what the fp16-row launch left.
// kFlush: as kWhole, in a step in which a tile leaves the window (plan.tiles_a is without it, the first of the row workgroups' tiles).
constexpr int kWhole = 0, kMixed = 1, kQuantisedRagged = 2, kFlush = 3;

// HP: head slots of a unit (2, 4 or 8).  CS: G > 32 (scales stored once per group of G = 32 << kg_shift).
template <int BITS, int HP, int MODE, bool CS>
__global__ __launch_bounds__(64 * kWaves, 3) void decode_tiles_kernel(TilesParams p) {
    constexpr bool kRagged = MODE == kQuantisedRagged;
    constexpr int kCodeBytes = kTileTokens * kHeadDim * BITS / 8;      // one tile of K or V codes
    constexpr int kPlanes = BITS / 2;
    constexpr int kScaleOff = 2 * kCodeBytes;                          // k_scale, k_zero, v_scale, v_zero: 256 bytes each
    constexpr int kSlotBytes = 2 * kCodeBytes + 1024;
    constexpr int NB = BITS == 2 ? 3 : 2;                              // tiles in flight per wavefront
    constexpr int NI = 2 * kPlanes + 1;                                // copy instructions per tile
    constexpr int NS = HP / 2;                                         // value-side operands per tile
    constexpr int HR = HP < 4 ? HP : BITS == 4 && HP == 8 ? 2 : 4;     // heads merged at once when a unit is left (LDS: three workgroups per compute unit)
    constexpr int kMaxParts = max_parts_of(BITS, HP);
    __shared__ __align__(16) unsigned char sm_ring[kWaves][NB][kSlotBytes];
    __shared__ __align__(16) float sm_o[kWaves][HR][kHeadDim];
    __shared__ __align__(16) unsigned char sm_q[2][HP < 4 ? 1024 : HP * 256];      // queries of this unit and the next
    __shared__ __align__(16) float sm_part[kRagged ? HP : 1][kHeadDim];              // the fp16-row launch's part of this unit
    __shared__ __align__(16) float sm_part_ml[kRagged ? HP : 1][4];                  // its (m, l, -, -) per head
    __shared__ float sm_ml[kWaves][HP][2];
    __shared__ int sm_last;

    static_assert(sizeof(sm_ring) + sizeof(sm_o) + sizeof(sm_q) + sizeof(sm_part) + sizeof(sm_part_ml) + sizeof(sm_ml) + 16 <= kLdsBytes, "occupancy");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kb = lane >> 4;
    const bool is_lo = n >= 8;
    const int head = n & (HP - 1);                                     // this lane's head slot
    const int kg = CS ? p.kg_shift : 0;
    // key tile rows: matrix row m holds token (m with its bits 2 and 3 exchanged) of its half-tile, so
    // that this lane's logits are those of tokens tok0 + i and 16 + tok0 + i, i = 0..3
    const int row_pos = (n & 3) | ((n >> 3) & 1) << 2 | ((n >> 2) & 1) << 3;
    const int tok0 = (kb & 1) * 8 + (kb >> 1) * 4;

    const int rep_total = p.n_q_heads / p.n_kv_heads, run = p.rep_here, n_runs = p.head_groups;
    auto kv_unit = [&](int u) -> int { return p.by_runs.of(u); };
    auto batch_of_kv = [&](int unit) -> int { return p.by_kv_heads.of(unit); };
    auto first_head = [&](int u) -> int {       // query head of head slot 0
        const int unit = kv_unit(u);
        return (unit - batch_of_kv(unit) * p.n_kv_heads) * rep_total + p.q_head0 + (u - unit * n_runs) * run;
    };
    auto live_heads = [&](int u) -> int { return min(run, rep_total - p.q_head0 - (u - kv_unit(u) * n_runs) * run); };
    auto batch_of = [&](int u) -> int { return batch_of_kv(kv_unit(u)); };

    // ---- this workgroup's interval of the axis of all-quantised steps ----
    const int tiles_a_plan = p.plan.tiles_a;
    const int n_a = (tiles_a_plan + kWaves - 1) / kWaves;              // steps per unit
    const int tiles_b = kRagged ? 0 : p.plan.tiles_total - tiles_a_plan;
    const int n_row_wgs = p.row_wgs;                                   // the first workgroups: fp16 rows, row_split per unit
    const int wg = (int)blockIdx.x - n_row_wgs;
    // The axis is one unit, cut into unit_wgs intervals (workgroup = unit * unit_wgs + interval), or, with unit_wgs = 0,
    // all units one after the other (kQuantisedRagged: always).
    const StepAxis axis{p.axis_len, p.axis_rem};
    const int unit_wgs = p.unit_wgs;
    // steps of a unit, and where they begin on the axis
    auto steps_of = [&](int u) -> int {
        if constexpr (kRagged) return ragged_steps(table(p.seq_state, 4 * batch_of(u)));
        else return n_a;                                               // (a sequence without quantised tiles has one empty step)
    };
    auto axis_start = [&](int u) -> int {
        if constexpr (kRagged) return table(p.unit_parts, batch_of(u)) + (u - batch_of(u) * p.n_kv_heads * n_runs) * steps_of(u);
        else return u * n_a;
    };
    // the workgroup's steps [j0, j1) in unit u, visited in an order rotated by the unit, so that workgroups in
    // lockstep do not all read the same relative offset of their units (which meets on few memory channels
    // for unlucky strides); `left`: steps of the interval not done yet
    struct Range { int j0, j1, at, tiles; };           // at: the step visited first
    auto range_of = [&](int u, int first, int left) -> Range {
        Range r;
        r.tiles = tiles_a_plan;
        if constexpr (kRagged) r.tiles = table(p.seq_state, 4 * batch_of(u)) / kTileTokens;
        r.j0 = first;
        r.j1 = min(steps_of(u), first + left);
        // (multiples of the golden ratio: neighbouring units start far apart)
        r.at = r.j0 + (int)(((uint64_t)((uint32_t)u * 0x9E3779B9u) * (uint32_t)(r.j1 - r.j0)) >> 32);
        return r;
    };

    // ---- copies of packed tiles into this wavefront's ring ----
    const uint32_t ring_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)&sm_ring[wave][0][0]);
    const uint32_t lane16 = lane * 16;
    // lanes 0-15 k_scale, 16-31 k_zero, 32-47 v_scale, 48-63 v_zero
    const __half* scale_base = kb == 0 ? p.k_scale : kb == 1 ? p.k_zero : kb == 2 ? p.v_scale : p.v_zero;
    const char* scale_lane = reinterpret_cast<const char*>(scale_base) + (CS && kb >= 2 ? min(n * 16, (256 >> kg) - 16) : n * 16);
    auto copy_tile = [&](int64_t tile, uint32_t dst) {
        const char* kc = reinterpret_cast<const char*>(p.k_codes) + tile * kCodeBytes;
        const char* vc = reinterpret_cast<const char*>(p.v_codes) + tile * kCodeBytes;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the slot's last readers have their data
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) copy_to_lds(kc + pl * 1024, lane16, dst + pl * 1024);
        int64_t off = tile * 256;
        if constexpr (CS) off = kb < 2 ? (tile >> kg) * 256 : (tile * 256) >> kg;
        copy_to_lds(scale_lane + off, dst + kScaleOff);
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) copy_to_lds(vc + pl * 1024, lane16, dst + kCodeBytes + pl * 1024);
    };
    // queries of unit u into sm_q[buf] (one instruction per 4 heads, by as many wavefronts)
    auto copy_query = [&](int u, int buf) {
        constexpr int kCopies = HP < 4 ? 1 : HP / 4;
        if (wave < kCopies) {
            const int row = min(wave * 4 + kb, live_heads(u) - 1);
            copy_to_lds(p.q + ((int64_t)batch_of(u) * p.n_q_heads + first_head(u) + row) * kHeadDim + n * 8,
                        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)&sm_q[buf][0]) + wave * 1024);
        }
    };

    // part 0 of unit u (what the fp16-row launch left) into LDS, to be there when the unit is left
    auto copy_rows_part = [&](int u) {
        const int live = live_heads(u);
        const int64_t prow = ((int64_t)batch_of(u) * p.n_q_heads + first_head(u)) * p.part_stride;
        constexpr int kCopies = (HP + 1) / 2;                           // two heads' outputs per instruction
        static_assert(kCopies <= kWaves, "one instruction per wavefront");
        if (wave < kCopies) {
            const int64_t row = prow + (int64_t)min(wave * 2 + (lane >> 5), live - 1) * p.part_stride;
            copy_to_lds(p.part_o + row * kHeadDim + (lane & 31) * 4, (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)&sm_part[wave * 2][0]));
        }
        if (wave == kWaves - 1 && lane < HP)
            copy_to_lds(p.part_ml + (prow + (int64_t)min(lane, live - 1) * p.part_stride) * 2,
                        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) float*)&sm_part_ml[0][0]));
    };

    // ---- per-wavefront state ----
    float4v acc[8];                    // value code sums: acc[u][i] = channel 16 u + 4 kb + i, column n
    float4v zsum;                      // value zero-point sums: zsum[i] = channel group i, column n
    float mref, l_lane;                // reference (log2 domain) of the probabilities; this lane's sum
    int ks;                            // value scales enter as s 2^-ks
    bool ks_set;
    uint32_t value_limit;              // fp16 pair: tiles with larger scales go to fit_value_exponent; below 2^(ks + kValueTop), or 0 with ks > 0
    half2v qz[4][4], qk[4][4];         // query: q 2^a; times 1 / position factor
    half2v rounded[4] = {};            // keys' products in the lo columns, 0 in the hi columns
    constexpr uint64_t kLoColumns = 0xFF00FF00FF00FF00ull;
    half2v q_zero[4];                  // HP < 8: q 2^a of channel block n / 4
    float c_code, c_zero;              // logit (log2 domain) = code sum * c_code + zero sum * c_zero

    auto reset_state = [&]() {
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8) acc[u8] = float4v{0.f, 0.f, 0.f, 0.f};
        zsum = float4v{0.f, 0.f, 0.f, 0.f};
        mref = -INFINITY;
        l_lane = 0.f;
        ks = 0;
        ks_set = false;
        value_limit = 0;
    };
    // query operands; raw[cb]: channels 32 cb + 8 kb .. + 7 of this lane's head (idle slots repeat the last head)
    auto set_query = [&](const half8 (&raw)[4]) {
        typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
        ushort2v top = {0, 0};                                          // |q| as integers
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                Frag f;
                f.h = raw[cb];
                top = __builtin_elementwise_max(top, __builtin_bit_cast(ushort2v, f.r[r] & 0x7FFF7FFFu));
            }
        float mx = (float)__builtin_bit_cast(_Float16, (unsigned short)max(top[0], top[1]));
        mx = max_rows(mx);
        const bool on = mx > 0.f;
        // 2^a mx in [2^8, 2^9) (a query below 2^-20 stays smaller), as two factors that fp16 holds
        const int a = on ? min(kQueryExp + 127 - (int)(__float_as_uint(mx) >> 23), 28) : 0, a1 = a / 2;
        const _Float16 up1 = on ? (_Float16)__uint_as_float((uint32_t)(127 + a1) << 23) : (_Float16)0.f;
        const _Float16 up2 = (_Float16)__uint_as_float((uint32_t)(127 + a - a1) << 23);
        const float down = p.softmax_scale * kLog2e * __uint_as_float((uint32_t)(127 - a) << 23);
        c_zero = down;
        c_code = down * kKeyUnscale;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            Frag f;
            f.h = raw[cb];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const _Float16 pf = BITS == 2 ? (_Float16)(1.f / (float)(1 << (2 * r))) : (_Float16)((r & 1) ? 1.f / 16.f : 1.f);
                qz[cb][r] = f.p[r] * half2v{up1, up1} * half2v{up2, up2};
                qk[cb][r] = qz[cb][r] * half2v{pf, pf};
            }
        }
        if constexpr (HP < 8) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const half2v even = is_lo ? qz[2][r] : qz[0][r], odd = is_lo ? qz[3][r] : qz[1][r];
                q_zero[r] = n & 4 ? odd : even;
            }
        }
    };

    // This lane's four sums of a tile out of the two half-tiles' results: the columns of a head share its 32
    // tokens, hi columns (n < 8) take tokens tok0 + i, lo columns tokens 16 + tok0 + i.
    auto own_half = [&](const float4v& d0, const float4v& d1, bool add_partner, float (&x)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            x[i] = is_lo ? d1[i] : d0[i];
            if (add_partner) x[i] += dpp<kDppRor8>(is_lo ? d0[i] : d1[i]);     // hi + lo column sum of that token
        }
    };
    // Probabilities p' = 2^(kProbExp + logit - mref) of this lane's four tokens; raises the reference
    // (and rescales the state: rescale(factor)) when a logit passes it by the slack.
    auto softmax = [&](const float (&x)[4], float cx, float zk, uint32_t live_mask, float (&pv)[4], auto&& rescale) {
        auto logits = [&](float off) {
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                pv[i] = fmaf(x[i], cx, off);
                if (!((live_mask >> i) & 1)) pv[i] = -INFINITY;
                mx = fmaxf(mx, pv[i]);
            }
            return mx;
        };
        const float mx = logits(zk - (mref - kProbExp<BITS>));
        if (__any(mx > (float)(kProbExp<BITS> + kSlack))) {
            const bool started = __any(mref != -INFINITY);
            float t = logits(zk);
            t = max_rows(fmaxf(t, dpp<kDppRor8>(t)));
            const float mnew = fmaxf(mref, t);
            const float f = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mnew);
            if (started) rescale(f);                   // (before, there is nothing to rescale)
            l_lane *= f;
            mref = mnew;
            logits(zk - (mref - kProbExp<BITS>));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) pv[i] = __builtin_amdgcn_exp2f(pv[i]);
        l_lane += (pv[0] + pv[1]) + (pv[2] + pv[3]);
    };
    auto rescale_acc = [&](float f) {
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8) acc[u8] *= f;
        zsum *= f;
    };

    // Value operand base: probabilities as fp16 hi + lo in the value tile's token order.
    // fb: hi (hi columns) or lo part (lo columns); fa: hi part in the lo columns, 0 in the others.
    auto split_probabilities = [&](const float (&pv)[4], Frag& fa, Frag& fb) {
        const half2v none = {(_Float16)0.f, (_Float16)0.f};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const half2v hi = pack_rtz(pv[2 * r], pv[2 * r + 1]);
            // the remainders (exact in fp32) with one mixed-precision instruction each
            float l0, l1;
            asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(l0) : "v"(hi), "v"(pv[2 * r]));
            asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(l1) : "v"(hi), "v"(pv[2 * r + 1]));
            const half2v lo = pack_rtz(l0, l1);
            // registers 0, 1: tokens tok0 + i (computed in the hi columns); 2, 3: 16 + tok0 + i (in the lo columns)
            fb.p[r] = from_partner<kLoLanes>(hi, lo);
            fb.p[r + 2] = from_partner<kHiLanes>(lo, hi);
            fa.p[r] = from_partner<kLoLanes>(none, hi);
            fa.p[r + 2] = is_lo ? hi : none;
        }
        // After the exchange of the upper half of registers 0, 1 with the lower half of 2, 3, lane kb holds
        // tokens 8 kb .. 8 kb + 7
        auto exchange = [&](Frag& f) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                auto s = __builtin_amdgcn_permlane32_swap(f.r[r], f.r[r + 2], false, false);
                f.r[r] = s[0];
                f.r[r + 2] = s[1];
            }
        };
        exchange(fa);
        exchange(fb);
    };

    // acc += codes x operand(p s); sv[set][r]: scales of the token pairs of this lane's channel group
    auto value_products = [&](const uint32_t* w, const half2v (&sv)[NS][4], Frag fa, Frag fb) {
        if constexpr (BITS == 2) {
            const half2v pf = {(_Float16)0.25f, (_Float16)0.25f};
            fa.p[1] *= pf; fa.p[3] *= pf;
            fb.p[1] *= pf; fb.p[3] *= pf;
        }
        Frag f[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const half2v t = fa.p[r] * sv[s][r];
                f[s].p[r] = __builtin_elementwise_fma(fb.p[r], sv[s][r], __builtin_elementwise_fma(fa.p[r], sv[s][r], -t));
            }
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8)
            acc[u8] = __builtin_amdgcn_mfma_f32_16x16x32_f16(value_fragment<BITS>(w, u8 >> 1, u8 & 1), f[(u8 >> 1) * NS / 4].h, acc[u8], 0, 0, 0);
    };
    // Exponent ks of the value scales (wave-uniform) that puts the largest of a tile's below 2^kValueTop; s2: two of them per lane
    auto wanted_exponent = [&](uint32_t s2) -> int {
        float mx = fmaxf((float)half2_of(s2)[0], (float)half2_of(s2)[1]);
        mx = max_rows(row_max(mx));
        const int e = (int)(__float_as_uint(mx) >> 23) - 126;              // mx < 2^e (mx = 0: e = -126)
        return __builtin_amdgcn_readfirstlane(max(e - kValueTop<BITS>, -24));
    };
    // two times the largest fp16 below 2^(k + kValueTop), at most the largest finite number
    auto top_scale = [&](int k) -> uint32_t {
        const int top = k + kValueTop<BITS> + 15;                           // biased fp16 exponent
        const uint32_t lim = top >= 31 ? 0x7BFFu : top <= 0 ? 0u : (uint32_t)(top << 10) - 1;
        return lim | lim << 16;
    };
    auto set_value_exponent = [&](int want) {
        if (ks_set) {
            const float f = __uint_as_float((uint32_t)(127 + ks - want) << 23);
#pragma unroll
            for (int u8 = 0; u8 < 8; ++u8) acc[u8] *= f;
        }
        ks = want;
        ks_set = true;
        value_limit = ks > 0 ? 0 : top_scale(ks);
    };
    auto max_pairs = [&](uint32_t a, uint32_t b) -> uint32_t {              // non-negative fp16 compare as integers
        typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2v, a), __builtin_bit_cast(ushort2v, b)));
    };
    auto any_above = [&](uint32_t s2, uint32_t limit) -> bool { return __any(max_pairs(s2, limit) != limit); };
    auto scale_values = [&](half2v (&sv)[NS][4]) {
        if (ks != 0) {
            // 2^-ks as two factors: each is a normal fp16 number for every ks in [-24, 16]
            const int k1 = ks / 2, k2 = ks - k1;
            const _Float16 f1 = (_Float16)__uint_as_float((uint32_t)(127 - k1) << 23), f2 = (_Float16)__uint_as_float((uint32_t)(127 - k2) << 23);
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) sv[s][r] = sv[s][r] * half2v{f1, f1} * half2v{f2, f2};
        }
    };

    // Fits ks to a tile: load(sv) reads its scales, s2: two of them per lane.  ks starts at 0, or lower where the unit's first
    // tile has small scales only.  It rises when a scale passes the limit AND its products with the probabilities are
    // large: a token with large values that nobody attends to must not take bits from the others of its tile.  It falls
    // back when all scales of a tile are far below the limit: nor from the tiles after it (value of 40 000 among values
    // of 1/16, probability 0: 3e-3 of the output when ks followed the scales alone).
    auto fit_value_exponent = [&](uint32_t s2, auto&& load, const Frag& fa, const Frag& fb) {
        if (!any_above(s2, value_limit)) return;
        bool high = true;
        if (ks > 0) {
            high = any_above(s2, top_scale(ks));
            if (!high && any_above(s2, (uint32_t)(ks + kValueTop<BITS> - kValueWindow + 15) * 0x04000400u)) return;
        }
        const int want = wanted_exponent(s2);
        int next = max(want, 0);
        if (high) {
            next = ks_set && ks >= 0 ? ks : want > -kValueWindow ? 0 : want;
            if (want > next) {
                half2v sv[NS][4];
                load(sv);
                float top = 0.f;
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const half2v p2 = is_lo ? fa.p[r] : fb.p[r];
                        top = fmaxf(top, fmaxf((float)p2[0] * (float)sv[s][r][0], (float)p2[1] * (float)sv[s][r][1]));
                    }
                if (__any(top > kValueProductLimit * __uint_as_float((uint32_t)(127 + next) << 23))) next = want;
            }
        }
        set_value_exponent(next);
    };

    // Raw key sums of a tile for this lane's four tokens; returns their factor.  big: the tile has scales past the limit.
    // Where the query makes such a channel's products leave fp16's range, all scales enter times 2^-kKeyScaleShift
    // for that head (small ones then lose bits, far below the large product); a channel that the query hardly
    // looks at costs the others nothing.
    auto key_products = [&](const uint32_t* w, Frag (&s)[4], bool big, float (&x)[4]) -> float {
        bool shift = false;
        if (big) {
            uint32_t top = kProductLimit;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) top = max_pairs(top, __builtin_bit_cast(uint32_t, qk[cb][r] * s[cb].p[r]) & 0x7FFF7FFFu);
            constexpr uint64_t kHeadLanes = HP == 8 ? 0x0101010101010101ull : HP == 4 ? 0x1111111111111111ull : 0x5555555555555555ull;
            int h = head;
            asm volatile("" : "+v"(h));                                    // (else the mask is kept in registers for all tiles)
            shift = (__builtin_amdgcn_ballot_w64(top != kProductLimit) & (kHeadLanes << h)) != 0;
            const _Float16 f1 = shift ? (_Float16)(1.f / (1 << kKeyScaleShift)) : (_Float16)1.f;
            const half2v f = {f1, f1};
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[cb].p[r] *= f;
        }
        float4v d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            Frag f;
            // In the lo columns alone; the hi columns' zeros stay.  (A second query with zeros there took sixteen registers, or was made
            // anew with twelve instructions a tile: 64 sequences of 500-8000 tokens, 32 / 8 heads 71.1 -> 70.1 us, 16 / 8 69.0 -> 67.1.)
            uint64_t active;
            asm("s_and_saveexec_b64 %4, %13\n\tv_pk_mul_f16 %0, %5, %9\n\tv_pk_mul_f16 %1, %6, %10\n\tv_pk_mul_f16 %2, %7, %11\n\tv_pk_mul_f16 %3, %8, %12\n\ts_mov_b64 exec, %4"
                : "+&v"(rounded[0]), "+&v"(rounded[1]), "+&v"(rounded[2]), "+&v"(rounded[3]), "=&s"(active)
                : "v"(qk[cb][0]), "v"(qk[cb][1]), "v"(qk[cb][2]), "v"(qk[cb][3]), "v"(s[cb].p[0]), "v"(s[cb].p[1]), "v"(s[cb].p[2]), "v"(s[cb].p[3]), "s"(kLoColumns)
                : "scc");
#pragma unroll
            for (int r = 0; r < 4; ++r) f.p[r] = __builtin_elementwise_fma(qk[cb][r], s[cb].p[r], -rounded[r]);
            d0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(key_fragment<BITS>(w, cb, 0), f.h, d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(key_fragment<BITS>(w, cb, 1), f.h, d1, 0, 0, 0);
        }
        own_half(d0, d1, true, x);
        return shift ? c_code * (float)(1 << kKeyScaleShift) : c_code;
    };
    auto query_frag = [&](int cb) -> half8 {
        Frag f;
#pragma unroll
        for (int r = 0; r < 4; ++r) f.p[r] = qz[cb][r];
        return f.h;
    };

    // value-side scale pairs of this lane's tokens 8 kb .. 8 kb + 7 out of an array [token][4] (or [token][4 >> kg]);
    // `at(byte)` reads four bytes at a byte offset of the tile's array
    const int my_group = HP == 2 ? (n >> 1) & 3 : HP == 4 ? (n >> 2) & 1 : 0;
    auto gather_pairs = [&](const unsigned char* base, int group, half2v (&out)[4]) {
        if constexpr (!CS) {
            const uint32_t sel = (group & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t t0 = *reinterpret_cast<const uint32_t*>(base + (kb * 8 + 2 * r) * 8 + (group >> 1) * 4);
                const uint32_t t1 = *reinterpret_cast<const uint32_t*>(base + (kb * 8 + 2 * r + 1) * 8 + (group >> 1) * 4);
                out[r] = half2_of(__builtin_amdgcn_perm(t1, t0, sel));
            }
        } else {
            const int per_token = 8 >> kg, off = (group >> kg) * 2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t t0 = *reinterpret_cast<const uint16_t*>(base + (kb * 8 + 2 * r) * per_token + off);
                const uint32_t t1 = *reinterpret_cast<const uint16_t*>(base + (kb * 8 + 2 * r + 1) * per_token + off);
                out[r] = half2_of(t0 | t1 << 16);
            }
        }
    };
    auto gather_scales = [&](const unsigned char* base, half2v (&sv)[NS][4]) {
        if constexpr (HP == 2 || CS) {
#pragma unroll
            for (int s = 0; s < NS; ++s) gather_pairs(base, HP == 2 ? my_group : HP == 4 ? 2 * s + my_group : s, sv[s]);
        } else {
            uint4v t[4];                                               // t[r]: tokens 2 r and 2 r + 1, four groups each
#pragma unroll
            for (int r = 0; r < 4; ++r) t[r] = *reinterpret_cast<const uint4v*>(base + kb * 64 + r * 16);
            if constexpr (HP == 4) {
                const uint32_t sel = my_group ? 0x07060302u : 0x05040100u;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sv[0][r] = half2_of(__builtin_amdgcn_perm(t[r][2], t[r][0], sel));
                    sv[1][r] = half2_of(__builtin_amdgcn_perm(t[r][3], t[r][1], sel));
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sv[0][r] = half2_of(__builtin_amdgcn_perm(t[r][2], t[r][0], 0x05040100u));
                    sv[1][r] = half2_of(__builtin_amdgcn_perm(t[r][2], t[r][0], 0x07060302u));
                    sv[2][r] = half2_of(__builtin_amdgcn_perm(t[r][3], t[r][1], 0x05040100u));
                    sv[3][r] = half2_of(__builtin_amdgcn_perm(t[r][3], t[r][1], 0x07060302u));
                }
            }
        }
    };
    // ---- one tile whose keys and values are all quantised, from an LDS slot ----
    // raw key sums x and the zero-points' share zk of the logits; returns the sums' factor
    auto slot_logits = [&](const unsigned char* sl, float (&x)[4], float& zk) -> float {
        uint32_t w[2 * BITS];
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) {
            const uint4v v = *reinterpret_cast<const uint4v*>(sl + pl * 1024 + (kb * 16 + row_pos) * 16);
            w[4 * pl + 0] = v[0]; w[4 * pl + 1] = v[1]; w[4 * pl + 2] = v[2]; w[4 * pl + 3] = v[3];
        }
        const bool big = any_above(*reinterpret_cast<const uint32_t*>(sl + kScaleOff + lane * 4), kKeyScaleLimit);
        float4v dz = {0.f, 0.f, 0.f, 0.f};
        Frag s[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            s[cb].h = *reinterpret_cast<const half8*>(sl + kScaleOff + cb * 64 + kb * 16);
            if constexpr (HP >= 8) {
                const half8 z = *reinterpret_cast<const half8*>(sl + kScaleOff + 256 + cb * 64 + kb * 16);
                dz = __builtin_amdgcn_mfma_f32_16x16x32_f16(z, query_frag(cb), dz, 0, 0, 0);
            }
        }
        if constexpr (HP < 8) {
            Frag z;
            z.h = *reinterpret_cast<const half8*>(sl + kScaleOff + 256 + (n >> 2) * 64 + kb * 16);
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) sum = __builtin_amdgcn_fdot2(q_zero[r], z.p[r], sum, false);
            sum += dpp<kDppRor8>(sum);
            sum += dpp<kDppRor4>(sum);
            dz[0] = add_rows(sum);
        }
        const float cx = key_products(w, s, big, x);
        zk = dz[0] * c_zero;
        return cx;
    };
    auto slot_scales = [&](const unsigned char* sl) -> uint32_t {          // two of the tile's value scales per lane
        return *reinterpret_cast<const uint32_t*>(sl + kScaleOff + 512 + (CS ? min(lane * 4, (256 >> kg) - 4) : lane * 4));
    };
    auto slot_outputs = [&](const unsigned char* sl, uint32_t s2, const float (&pv)[4]) {
        Frag fa, fb, z;
        split_probabilities(pv, fa, fb);
        fit_value_exponent(s2, [&](half2v (&to)[NS][4]) { gather_scales(sl + kScaleOff + 512, to); }, fa, fb);
        half2v sv[NS][4];
        gather_scales(sl + kScaleOff + 512, sv);
        gather_pairs(sl + kScaleOff + 768, n & 3, z.p);
        zsum = __builtin_amdgcn_mfma_f32_16x16x32_f16(z.h, fb.h, zsum, 0, 0, 0);      // rows = channel groups
        scale_values(sv);
        uint32_t w[2 * BITS];
#pragma unroll
        for (int pl = 0; pl < kPlanes; ++pl) {
            const uint4v v = *reinterpret_cast<const uint4v*>(sl + kCodeBytes + pl * 1024 + lane16);
            w[4 * pl + 0] = v[0]; w[4 * pl + 1] = v[1]; w[4 * pl + 2] = v[2]; w[4 * pl + 3] = v[3];
        }
        value_products(w, sv, fa, fb);
    };
    auto quantised_tile = [&](const unsigned char* sl) {
        float x[4], pv[4], zk;
        const float cx = slot_logits(sl, x, zk);
        const uint32_t s2 = slot_scales(sl);
        softmax(x, cx, zk, 0xfu, pv, rescale_acc);
        slot_outputs(sl, s2, pv);
    };

    // ---- fp16 rows of a tile: keys as matrix operands, values for the fp32 products ----
    // key rows: half-tile b2, row row_pos; value rows: the tokens whose probabilities the lane holds, channels 8 n ..
    // (rows past the end re-read the last row and are masked; the newest token may not be in the rings yet)
    auto load_key_rows = [&](int64_t unit, int tt, half8 (&kr)[2][4]) {
        const int last = p.length - 1;
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
            const int t = min(tt + b2 * 16 + row_pos, last);
            const __half* src = p.k_new && t == last ? p.k_new + unit * kHeadDim
                                                     : p.k_resid + (unit * p.cap_r + ring_slot(p.k_r_start, t - p.n_kq, p.cap_r)) * kHeadDim;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) kr[b2][cb] = *reinterpret_cast<const half8*>(src + cb * 32 + kb * 8);
        }
    };
    auto load_value_rows = [&](int64_t unit, int tt, half8 (&vr)[8]) {
        const int last = p.length - 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = min(max(tt + (i >> 2) * 16 + tok0 + (i & 3), p.n_vq), last);
            const __half* src = p.v_new && t == last ? p.v_new + unit * kHeadDim
                                                     : p.v_resid + (unit * p.cap_r + ring_slot(p.v_r_start, t - p.n_vq, p.cap_r)) * kHeadDim;
            vr[i] = *reinterpret_cast<const half8*>(src + n * 8);
        }
    };
    // the query's columns hold the same head twice, so hi and lo column agree and nothing is added up
    auto row_logits = [&](const half8 (&kr)[2][4], float (&x)[4]) {
        float4v d[2];
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
            d[b2] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) d[b2] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kr[b2][cb], query_frag(cb), d[b2], 0, 0, 0);
        }
        own_half(d[0], d[1], false, x);
    };
    // a 16x16x4 fp32 product takes one token of each kb and element e of every lane: ro[e], row 4 kb + i ->
    // channel 8 (4 kb + i) + e, column n (hi columns; the lo columns are not used)
    auto row_outputs = [&](const half8 (&vr)[8], const float (&pr)[4], float4v (&ro)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float p0 = pr[i], p1 = dpp<kDppRor8>(pr[i]);             // tokens tok0 + i and 16 + tok0 + i (hi columns)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ro[e] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)vr[i][e], p0, ro[e], 0, 0, 0);
                ro[e] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)vr[4 + i][e], p1, ro[e], 0, 0, 0);
            }
        }
    };
    // the heads [h0, h0 + count) of ro as rows of 128 channels
    auto store_rows = [&](const float4v (&ro)[8], float (*rows)[kHeadDim], int h0, int count) {
        if (n >= h0 && n < h0 + count) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float* dst = &rows[n - h0][(kb * 4 + i) * 8];
                *reinterpret_cast<float4v*>(dst) = float4v{ro[0][i], ro[1][i], ro[2][i], ro[3][i]};
                *reinterpret_cast<float4v*>(dst + 4) = float4v{ro[4][i], ro[5][i], ro[6][i], ro[7][i]};
            }
        }
    };
    // fused append: the wavefront that owns the newest token's tile stores its rows in the rings
    // (lanes 0-15 the key row, 16-31 the value row); every reader of that token takes it from k_new / v_new
    auto append_new_token = [&](int u, int tile) {
        const int last = p.length - 1;
        if (p.k_new && tile == last / kTileTokens && lane < 32 && u == kv_unit(u) * n_runs && p.q_head0 == 0) {
            const int64_t unit = kv_unit(u);
            const bool is_v = lane >= 16;
            const int ring = is_v ? ring_slot(p.v_r_start, last - p.n_vq, p.cap_r) : ring_slot(p.k_r_start, last - p.n_kq, p.cap_r);
            const uint4v v = *reinterpret_cast<const uint4v*>((is_v ? p.v_new : p.k_new) + unit * kHeadDim + n * 8);
            *reinterpret_cast<uint4v*>(const_cast<__half*>(is_v ? p.v_resid : p.k_resid) + (unit * p.cap_r + ring) * kHeadDim + n * 8) = v;
        }
    };
    // one tile that holds fp16 rows, or in which K and V are split differently: what is packed of it goes through an LDS
    // slot like any other tile (reading its scales one by one into registers instead took 1.3 times as long, 1.5 times
    // with G > 32: 64 x 32 / 8 heads, 1500 tokens, Algorithm 1's policy)
    auto general_tile = [&](int u, int tile) {
        const int64_t unit = kv_unit(u);
        const int tt = tile * kTileTokens, last = p.length - 1;
        unsigned char* sl = &sm_ring[wave][0][0];
        float x[4], pv[4];
        float zk = 0.f, cx = c_zero;
        const int tok = tok0 + (is_lo ? 16 : 0);                       // this lane's tokens: tok + i
        const int n_vq_here = min(max(p.n_vq - tt, 0), kTileTokens);
        if (tt < p.n_kq || n_vq_here > 0) {                             // (the tile lies within the packed arrays' capacity)
            copy_tile(unit * p.cap_tiles + tile, ring_lds);
            wait_copies<0>();
        }
        if (tt < p.n_kq) {
            cx = slot_logits(sl, x, zk);
        } else {
            half8 kr[2][4];
            load_key_rows(unit, tt, kr);
            row_logits(kr, x);
        }
        uint32_t live = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) live |= (tt + tok + i <= last ? 1u : 0u) << i;
        softmax(x, cx, zk, live, pv, rescale_acc);
        if (n_vq_here > 0) {
            if (n_vq_here < kTileTokens) {
                // scales and zero-points of tokens that are not quantised yet may hold anything: 0
                const int per_token = CS ? 4 >> kg : 4;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int at = 2 * lane + i;
                    if (at < kTileTokens * per_token && at >= n_vq_here * per_token) {
                        reinterpret_cast<uint16_t*>(sl + kScaleOff + 512)[at] = 0;
                        reinterpret_cast<uint16_t*>(sl + kScaleOff + 768)[at] = 0;
                    }
                }
                wave_lds_sync();
            }
            float pq[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pq[i] = tok + i < n_vq_here ? pv[i] : 0.f;
            slot_outputs(sl, slot_scales(sl), pq);
        }
        if (n_vq_here < kTileTokens && p.n_vr > 0) {
            // (rows in LDS: the rest of the ring)
            float (*rows)[kHeadDim] = reinterpret_cast<float (*)[kHeadDim]>(&sm_ring[wave][1][0]);
            static_assert(sizeof(float) * HP * kHeadDim <= (NB - 1) * kSlotBytes, "one row per head");
            const float f = __uint_as_float((uint32_t)(127 - ks) << 23) * (1.0f / kValueUnscale);
            half8 vr[8];
            load_value_rows(unit, tt, vr);
            float pr[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pr[i] = tok + i >= n_vq_here ? pv[i] : 0.f;        // 0 past the end already
            float4v ro[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) ro[e] = float4v{0.f, 0.f, 0.f, 0.f};
            row_outputs(vr, pr, ro);
            wave_lds_sync();
            store_rows(ro, rows, 0, HP);
            wave_lds_sync();
            if (!is_lo) {
#pragma unroll
                for (int u8 = 0; u8 < 8; ++u8) acc[u8] += *reinterpret_cast<const float4v*>(&rows[head][u8 * 16 + kb * 4]) * f;
            }
            wave_lds_sync();
        }
        append_new_token(u, tile);
    };

    // ---- leave a unit: merge the four wavefronts; write the output or this workgroup's part ----
    // rows: this workgroup holds fp16 rows of the unit (the first parts), otherwise some of its all-quantised steps
    // last: of the workgroup, so that no copies are in flight and all heads' outputs fit the rings; otherwise HR heads at a time
    // write_o(o, h0, count, f): this wavefront's outputs of the heads [h0, h0 + count), times f, as rows from o on
    auto leave_unit = [&](int u, bool rows, bool last, auto&& write_o) {
        const int64_t row0 = (int64_t)batch_of(u) * p.n_q_heads + first_head(u);
        const int live = live_heads(u);
        int parts = 0, mine = 0;
        const int steps = steps_of(u);
        if (!kRagged && unit_wgs > 0) {
            parts = unit_wgs;
            mine = wg - u * unit_wgs;
        } else if (steps > 0) {
            const int at = axis_start(u), g0 = axis.owner(at, p.by_axis_longer, p.by_axis_len);
            parts = axis.owner(at + steps - 1, p.by_axis_longer, p.by_axis_len) - g0 + 1;
            mine = wg - g0;
        }
        if (tiles_b > 0) {
            parts += p.row_split;
            mine = rows ? (int)blockIdx.x - p.by_row_split.of(blockIdx.x) * p.row_split : mine + p.row_split;
        }
        const int stride = p.part_stride, base = kRagged ? 1 : 0;           // part 0: the fp16-row launch's
        // the wavefronts' statistics, then their outputs relative to the common maximum
        {
            const float l = add_rows(l_lane + dpp<kDppRor8>(l_lane));
            if (lane < HP) {
                sm_ml[wave][lane][0] = mref;
                sm_ml[wave][lane][1] = l;
            }
        }
        lds_barrier();
        float m_all = -INFINITY;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) m_all = fmaxf(m_all, sm_ml[w][head][0]);
        const float f_own = mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - m_all);
        static_assert(HP * kHeadDim * sizeof(float) <= sizeof(sm_ring[0]), "all heads' outputs");
        const int at_once = last ? HP : HR;
        const uint32_t o_stride = last ? sizeof(sm_ring[0]) / sizeof(float) : HR * kHeadDim;      // from wavefront to wavefront
        float* o_base = last ? reinterpret_cast<float*>(&sm_ring[0][0][0]) : &sm_o[0][0][0];
#pragma unroll 1
        for (int h0 = 0; h0 < HP; h0 += at_once) {
            write_o(o_base + wave * o_stride, h0, at_once, f_own);
            lds_barrier();
            const int c = tid % (kHeadDim / 2) * 2;                                     // two channels of one head
#pragma unroll 1
            for (int hh = h0 + tid / (kHeadDim / 2); hh < min(h0 + at_once, live); hh += kWaves) {
                float m = -INFINITY, ll = 0.f;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) m = fmaxf(m, sm_ml[w][hh][0]);
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const float mw = sm_ml[w][hh][0];
                    ll = fmaf(sm_ml[w][hh][1], mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - m), ll);
                }
                m -= (float)kProbExp<BITS>;                                // o and l are relative to 2^m
                float2 oo = {0.f, 0.f};
#pragma unroll
                for (int w = 0; w < kWaves; ++w) {
                    const float2 x = *reinterpret_cast<const float2*>(o_base + w * o_stride + (hh - h0) * kHeadDim + c);
                    oo.x += x.x;
                    oo.y += x.y;
                }
                const int64_t prow = (row0 + hh) * stride;
                if (parts == 1) {
                    if constexpr (kRagged) {
                        const float mr = sm_part_ml[hh][0], mn = fmaxf(m, mr);        // the fp16-row launch's part
                        const float f0 = __builtin_amdgcn_exp2f(m - mn), f1 = __builtin_amdgcn_exp2f(mr - mn);
                        oo.x = fmaf(oo.x, f0, sm_part[hh][c] * f1);
                        oo.y = fmaf(oo.y, f0, sm_part[hh][c + 1] * f1);
                        ll = fmaf(ll, f0, sm_part_ml[hh][1] * f1);
                    }
                    *reinterpret_cast<float2*>(p.out + (row0 + hh) * kHeadDim + c) = make_float2(oo.x / ll, oo.y / ll);
                } else {
                    const int64_t at = prow + base + mine;
                    device_store(p.part_o + at * kHeadDim + c, oo);
                    if (c == 0) device_store(p.part_ml + at * 2, make_float2(m, ll));
                }
            }
            if (h0 + at_once < HP || parts == 1) lds_barrier();            // LDS is written again
        }
        if (parts > 1) {
            // published as in decode_mfma_kernel: device-scope stores, the wait for their acknowledgement,
            // the barrier, then the unit's counter; the last workgroup merges
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();
            if (tid == 0) {
                const int done = __hip_atomic_fetch_add(p.counters + u, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                sm_last = done == parts - 1;
            }
            lds_barrier();
            if (sm_last) {
                // Outputs: one thread per head and four channels; with fewer than eight heads the threads share a head's
                // parts, kBatch consecutive ones at a time.  Statistics: 32 threads per head.  All first loads are in
                // flight together: one trip to memory for up to kBatch * kShares parts.
                constexpr int kQuads = HP * kHeadDim / 4, kShares = 64 * kWaves / kQuads;
                constexpr int kBatch = kShares == 1 ? 24 : kShares == 2 ? 16 : 12, kRound = kBatch * kShares;
                constexpr int kPad = (kMaxParts + kRound - 1) / kRound * kRound;
                float (*sm_w)[kPad] = reinterpret_cast<float (*)[kPad]>(&sm_o[0][0][0]);       // weights, 0 past the last part
                static_assert(sizeof(float) * HP * kPad <= sizeof(sm_o) && sizeof(sm_o) >= 16 * 64 * kWaves && kShares <= kWaves, "LDS of the merge");
                const int quad = tid % kQuads, share = __builtin_amdgcn_readfirstlane(tid / kQuads), hh = quad / (kHeadDim / 4), c = quad % (kHeadDim / 4) * 2;
                const float* po = p.part_o + ((row0 + min(hh, live - 1)) * stride + base) * kHeadDim + c;
                uint64_t ov[kBatch][2];
                load_parts(po, share * kBatch, parts, ov);
                const int sh = tid / 32, sp = tid % 32;
                if (sh < HP) {
                    constexpr int kStat = (kMaxParts + 31) / 32;
                    float2 v[kStat];
                    const float* ml = p.part_ml + ((row0 + min(sh, live - 1)) * stride + base) * 2;
#pragma unroll
                    for (int k = 0; k < kStat; ++k) {
                        v[k] = make_float2(-INFINITY, 0.f);
                        if (32 * k < parts)
                            v[k] = __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(ml + 2 * min(sp + 32 * k, parts - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    }
                    float m = kRagged ? sm_part_ml[min(sh, live - 1)][0] : -INFINITY;
#pragma unroll
                    for (int k = 0; k < kStat; ++k) m = fmaxf(m, v[k].x);
                    m = half_max(m);
                    float lsum = 0.f;
#pragma unroll
                    for (int k = 0; k < kStat; ++k) {
                        const int i = sp + 32 * k;
                        const float w = i < parts && v[k].x != -INFINITY ? __builtin_amdgcn_exp2f(v[k].x - m) : 0.f;
                        lsum = fmaf(v[k].y, w, lsum);
                        if (i < kPad) sm_w[sh][i] = w;
                    }
#pragma unroll
                    for (int i = sp + 32 * kStat; i < kPad; i += 32) sm_w[sh][i] = 0.f;
                    lsum = half_sum(lsum);
                    if (sp == 0) {
                        if constexpr (kRagged) {
                            const float w = __builtin_amdgcn_exp2f(sm_part_ml[min(sh, live - 1)][0] - m);
                            lsum = fmaf(sm_part_ml[min(sh, live - 1)][1], w, lsum);
                            sm_ml[1][sh][0] = w;
                        }
                        sm_ml[0][sh][0] = lsum;
                    }
                }
                lds_barrier();
                float4v o = {0.f, 0.f, 0.f, 0.f};
                for (int i0 = share * kBatch; i0 < parts; i0 += kRound) {
                    if (i0 != share * kBatch) load_parts(po, i0, parts, ov);
#pragma unroll
                    for (int j = 0; j < kBatch; ++j) {
                        const float w = sm_w[hh][i0 + j];
                        const float2 oa = __builtin_bit_cast(float2, ov[j][0]), ob = __builtin_bit_cast(float2, ov[j][1]);
                        o += float4v{oa.x, oa.y, ob.x, ob.y} * w;
                    }
                }
                if constexpr (kRagged) {
                    if (share == 0) {
                        const float2 oa = *reinterpret_cast<const float2*>(&sm_part[hh][c]), ob = *reinterpret_cast<const float2*>(&sm_part[hh][c + 64]);
                        o += float4v{oa.x, oa.y, ob.x, ob.y} * sm_ml[1][hh][0];
                    }
                }
                if constexpr (kShares > 1) {                            // add up the shares
                    lds_barrier();                                      // (the weights have been read)
                    float4v* sums = reinterpret_cast<float4v*>(&sm_o[0][0][0]);
                    sums[tid] = o;
                    lds_barrier();
                    if (share == 0) {
                        o = sums[quad];
#pragma unroll
                        for (int s2 = 1; s2 < kShares; ++s2) o += sums[s2 * kQuads + quad];
                    }
                }
                if (share == 0 && hh < live) {
                    float* dst = p.out + (row0 + hh) * kHeadDim + c;
                    o /= sm_ml[0][hh][0];
                    *reinterpret_cast<float2*>(dst) = make_float2(o[0], o[1]);
                    *reinterpret_cast<float2*>(dst + 64) = make_float2(o[2], o[3]);
                }
                if (tid == 0) __hip_atomic_store(p.counters + u, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            lds_barrier();
        }
    };

    auto write_acc = [&](float* rows, int h0, int count, float f) {
        float zz[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) zz[g] = (zsum[g] + dpp<kDppRor8>(zsum[g])) * f;
        const float up = kValueUnscale * __uint_as_float((uint32_t)(127 + ks) << 23) * f;
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8) {
            const int g = u8 >> 1;
            float4v o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = fmaf(acc[u8][i] + dpp<kDppRor8>(acc[u8][i]), up, zz[g]);
            const bool valid = !is_lo && (HP == 8 || (HP == 4 ? my_group == (g & 1) : my_group == g));
            if (valid && head >= h0 && head < h0 + count) *reinterpret_cast<float4v*>(rows + (head - h0) * kHeadDim + u8 * 16 + kb * 4) = o;
        }
    };

    if constexpr (MODE == kWhole || MODE == kFlush) {
        if (wg < 0) {                                  // ---- the fp16 rows of one unit (K and V split alike) ----
            constexpr int kFlushed = MODE == kFlush ? 1 : 0;
            const int u = p.by_row_split.of(blockIdx.x), cut = (int)blockIdx.x - u * p.row_split;
            // kFlush: the first one's last wavefront quantises the tile that leaves the window and attends to it, the others have the rows
            const bool flushes = kFlushed && cut == 0 && wave == kWaves - 1;
            const int tile0 = flushes ? p.plan.tiles_total : tiles_a_plan + cut * kWaves + wave + (cut > 0 ? 0 : kFlushed);
            const int64_t unit = kv_unit(u);
            half8 raw[4], kr[2][4], vr[8];
            const int live = live_heads(u), last = p.length - 1;
            const __half* src = p.q + ((int64_t)batch_of(u) * p.n_q_heads + first_head(u) + min(head, live - 1)) * kHeadDim + kb * 8;
            float4v ro[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) ro[e] = float4v{0.f, 0.f, 0.f, 0.f};
            mref = -INFINITY;
            l_lane = 0.f;
            if constexpr (MODE == kFlush) {
                if (flushes) {
                    unsigned char* sl = &sm_ring[wave][0][0];
                    tile::flush_tile<BITS>(p, unit, unit * p.cap_tiles + tiles_a_plan, lane, sl, u == kv_unit(u) * n_runs && p.q_head0 == 0);
                    wave_lds_sync();
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb) raw[cb] = *reinterpret_cast<const half8*>(src + cb * 32);
                    reset_state();
                    set_query(raw);
                    quantised_tile(sl);
                }
            }
            for (int tile = tile0; tile < p.plan.tiles_total; tile += kWaves * p.row_split - kFlushed) {
                const int tt = tile * kTileTokens, tok = tok0 + (is_lo ? 16 : 0);
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) raw[cb] = *reinterpret_cast<const half8*>(src + cb * 32);
                load_key_rows(unit, tt, kr);
                load_value_rows(unit, tt, vr);
                set_query(raw);
                float x[4], pv[4];
                row_logits(kr, x);
                uint32_t alive = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) alive |= (tt + tok + i <= last ? 1u : 0u) << i;
                softmax(x, c_zero, 0.f, alive, pv, [&](float f) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) ro[e] *= f;
                });
                row_outputs(vr, pv, ro);
                append_new_token(u, tile);
            }
            leave_unit(u, true, true, [&](float* to, int h0, int count, float f) {
                if (flushes) {
                    write_acc(to, h0, count, f);
                    return;
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) ro[e] *= f;
                store_rows(ro, reinterpret_cast<float (*)[kHeadDim]>(to), h0, count);
            });
            return;
        }
    }
    if constexpr (MODE == kMixed) {
        if (wg < 0) {                                  // ---- the tiles of one unit that hold fp16 rows or are split differently ----
            const int u = p.by_row_split.of(blockIdx.x), tile0 = tiles_a_plan + ((int)blockIdx.x - u * p.row_split) * kWaves + wave;
            half8 raw[4];
            const int live = live_heads(u);
            const __half* src = p.q + ((int64_t)batch_of(u) * p.n_q_heads + first_head(u) + min(head, live - 1)) * kHeadDim + kb * 8;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) raw[cb] = *reinterpret_cast<const half8*>(src + cb * 32);
            reset_state();
            set_query(raw);
            for (int tile = tile0; tile < p.plan.tiles_total; tile += kWaves * p.row_split) general_tile(u, tile);
            leave_unit(u, true, true, write_acc);
            return;
        }
    }

    // ---- all-quantised steps ----
    int u, first, left;
    if constexpr (kRagged) {
        u = table(p.wave_desc, 4 * wg + 0);
        first = table(p.wave_desc, 4 * wg + 1);
        left = table(p.wave_desc, 4 * wg + 2);
    } else if (unit_wgs > 0) {
        u = p.by_unit_wgs.of(wg);
        const int g = wg - u * unit_wgs;
        first = axis.start(g);
        left = axis.start(g + 1) - first;
    } else {
        const int pos0 = axis.start(wg);
        u = p.by_steps.of(pos0);
        first = pos0 - u * n_a;
        left = axis.start(wg + 1) - pos0;
    }
    copy_query(u, 0);
    // cursor of the next tile to copy: the interval's steps, unit by unit
    // (No divisions after a copy: 130 scalar instructions a tile then, 40 now; launches 0.7-1 us shorter.)
    Range nx = range_of(u, first, left);
    int nx_u = u, nx_here = nx.j1 - nx.j0, nx_left = left;            // steps left in this unit, and in all
    int64_t nx_tile0 = (int64_t)kv_unit(u) * p.cap_tiles;
    uint32_t nx_dst = ring_lds;
    auto advance_copy = [&]() {
        if (nx_left <= 0) return;
        copy_tile(nx_tile0 + max(min(nx.at * kWaves + wave, nx.tiles - 1), 0), nx_dst);
        nx_dst = nx_dst == ring_lds + (NB - 1) * kSlotBytes ? ring_lds : nx_dst + kSlotBytes;
        nx.at = nx.at + 1 == nx.j1 ? nx.j0 : nx.at + 1;
        --nx_left;
        if (--nx_here == 0 && nx_left > 0) {
            ++nx_u;
            nx = range_of(nx_u, 0, nx_left);
            nx_here = nx.j1 - nx.j0;
            nx_tile0 = (int64_t)kv_unit(nx_u) * p.cap_tiles;
        }
    };
    // waits for the oldest of the tiles in flight: `todo` steps are left, so min(todo, NB) tiles are in flight
    auto wait_oldest = [&](int todo) {
        if (todo >= NB) wait_copies<(NB - 1) * NI>();
        else if (NB > 2 && todo == 2) wait_copies<NI>();
        else wait_copies<0>();
    };
    // One tile at first, the others when the query is ready: the first NB tiles of all wavefronts together keep the memory busy for
    // 4-5 us, and with all of them asked for at once the first ones came that late (after 7.1 us, now 5.3: 64 / 8 heads, batch 4,
    // 16 377 tokens 30.1 -> 29.5 us, 32 / 8 heads, 32 767 tokens 31.2 -> 30.2, 71 / 1 heads 29.4 -> 28.2).
    advance_copy();
    wait_copies<NI>();                                 // the query has arrived, the tile is on its way
    lds_barrier();
    int slot = 0, q_buf = 0, ahead = 1;
    // The instruction arbiter favours the oldest wavefront of a SIMD, so the workgroups of a compute unit
    // would finish one after the other, the last one alone and latency-bound: a wavefront's priority falls with
    // the share of its interval that is done.
    const int quarter = left >> 2;
    int priority = 3, drop_at = 3 * quarter;
    __builtin_amdgcn_s_setprio(3);
    auto set_progress_priority = [&](int remaining) {
        if (remaining > drop_at) return;
        --priority;
        drop_at -= quarter;
        if (priority == 2) __builtin_amdgcn_s_setprio(2);
        else if (priority == 1) __builtin_amdgcn_s_setprio(1);
        else {
            __builtin_amdgcn_s_setprio(0);
            drop_at = 0;
        }
    };
#pragma unroll 1
    while (true) {
        const Range r = range_of(u, first, left);
        int at = r.at;
        left -= r.j1 - r.j0;
        {
            half8 raw[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) raw[cb] = *reinterpret_cast<const half8*>(&sm_q[q_buf][min(head, live_heads(u) - 1) * 256 + cb * 64 + kb * 16]);
            reset_state();
            set_query(raw);
        }
#pragma unroll 1
        for (; ahead < NB; ++ahead) advance_copy();
        if (left > 0) copy_query(u + 1, q_buf ^ 1);
        if constexpr (kRagged) copy_rows_part(u);
        for (int j = r.j0; j < r.j1; ++j) {
            const int todo = left + r.j1 - j;          // steps of the interval that are not done
            set_progress_priority(todo);
            wait_oldest(todo);
            if (at * kWaves + wave < r.tiles) quantised_tile(&sm_ring[wave][slot][0]);
            advance_copy();
            at = at + 1 == r.j1 ? r.j0 : at + 1;
            slot = slot + 1 == NB ? 0 : slot + 1;
        }
        // the next query and the rows' part: there already if a tile requested after them was waited for
        if ((kRagged || left > 0) && r.j1 - r.j0 <= NB) wait_copies<0>();
        leave_unit(u, false, left <= 0, write_acc);                          // (its barriers make the query visible to all wavefronts)
        if (left <= 0) break;
        ++u;
        first = 0;
        q_buf ^= 1;
    }
    wait_copies<0>();                                  // no copy may land in LDS that has been given back
}

constexpr int kMaxDevices = 64;
// workgroups the current device holds at once (an occupancy query, kept per device)
template <int BITS, int HP, int MODE, bool CS>
int resident_workgroups() {
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256 * 3;
    const bool keep = dev >= 0 && dev < kMaxDevices;
    if (keep) {
        const int c = cached[dev].load(std::memory_order_relaxed);
        if (c > 0) return c;
    }
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_tiles_kernel<BITS, HP, MODE, CS>, 64 * kWaves, 0) != hipSuccess ||
        cus <= 0 || per_cu <= 0)
        return 256 * 3;
    if (keep) cached[dev].store(cus * per_cu, std::memory_order_relaxed);
    return cus * per_cu;
}

// fn<BITS, HP>() for the head slots that hold `rep` query heads
template <class F>
bool with_tiles_variant(int bits, int rep, F&& fn) {
    const int hp = rep <= 2 ? 2 : rep <= 4 ? 4 : 8;
    if (rep > 8 || rep < 1) return false;
#define KIVI_TILES(B, H) if (bits == B && hp == H) { fn(std::integral_constant<int, B>{}, std::integral_constant<int, H>{}); return true; }
    KIVI_TILES(2, 2) KIVI_TILES(2, 4) KIVI_TILES(2, 8)
    KIVI_TILES(4, 2) KIVI_TILES(4, 4) KIVI_TILES(4, 8)
#undef KIVI_TILES
    return false;
}

template <int BITS, int HP, int MODE, bool CS>
hipError_t launch_mode(const DecodeParams& params, hipStream_t stream) {
    TilesParams p{};
    static_cast<DecodeParams&>(p) = params;
    const int64_t units = (int64_t)p.batch * p.n_kv_heads * p.head_groups;
    p.by_runs = FastDiv::by(p.head_groups);
    p.by_kv_heads = FastDiv::by(p.n_kv_heads);
    auto set_axis = [&]() {
        p.by_axis_len = FastDiv::by(p.axis_len);
        p.by_axis_longer = FastDiv::by(p.axis_len + 1);
    };
    if constexpr (MODE == kQuantisedRagged) {
        set_axis();
        if (p.n_slices < 1 || !p.wave_desc || !p.unit_parts || !p.seq_state) return hipErrorInvalidValue;
        p.row_wgs = 0;
        decode_tiles_kernel<BITS, HP, MODE, CS><<<p.n_slices, 64 * kWaves, 0, stream>>>(p);
        return hipGetLastError();
    }
    UniformCut cut;
    const bool two = p.two_launches > 0 && p.plan.tiles_total > p.plan.tiles_a && p.plan.tiles_a > 0;      // the fp16 rows in a launch of their own
    // (kFlush: no further row workgroup for the flushed tile's sake -- one more part to merge: 32 units x 2047, 4 bits, 16.6 us with,
    // 14.7 without)
    if (!cut_uniform(units, p.plan.tiles_a, p.plan.tiles_total - (MODE == kFlush ? 1 : 0), resident_workgroups<BITS, HP, MODE, CS>(), p.part_stride, max_parts_of(BITS, HP), two, p.rows_for_tiles, cut))
        return hipErrorInvalidValue;
    p.row_split = cut.row_split;
    p.row_wgs = cut.row_wgs;
    p.unit_wgs = cut.unit_wgs;
    p.axis_len = cut.axis.len;
    p.axis_rem = cut.axis.rem;
    set_axis();
    p.by_row_split = FastDiv::by(cut.row_split);
    p.by_unit_wgs = FastDiv::by(std::max(cut.unit_wgs, 1));
    p.by_steps = FastDiv::by(std::max((p.plan.tiles_a + kWaves - 1) / kWaves, 1));
    if (p.rows_for_tiles) {
        if (!two) return hipErrorInvalidValue;
        p.row_wgs = 0;
    } else if (two) {
        decode_tiles_kernel<BITS, HP, MODE, CS><<<(unsigned)p.row_wgs, 64 * kWaves, 0, stream>>>(p);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        p.row_wgs = 0;
    }
    decode_tiles_kernel<BITS, HP, MODE, CS><<<(unsigned)(cut.intervals + p.row_wgs), 64 * kWaves, 0, stream>>>(p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode_tiles(DecodeParams p, hipStream_t stream) {
    const int rep_total = p.n_q_heads / p.n_kv_heads;
    if (p.head_groups < 1 || p.rep_here < 1 || (p.head_groups > 1 && (p.q_head0 != 0 || p.head_groups * p.rep_here < rep_total || (p.head_groups - 1) * p.rep_here >= rep_total)))
        return hipErrorInvalidValue;
    if (p.seq_state) {
        if (p.k_new || p.flush_k || p.two_launches == 0) return hipErrorInvalidValue;      // (launch_ragged_rows goes before)
    }
    const bool flush_inside = p.flush_k && p.flush_v && p.two_launches == 0;
    if (flush_inside) {
        // one tile, the last quantised one, out of the rings right before the window: the row workgroups' first
        if (p.seq_state || p.kg_shift > 0 || p.n_kq != p.n_vq || p.n_kr < 1 || p.plan.tiles_a < 1 || p.flush_k->n_tiles != 1 || p.flush_v->n_tokens != kTileTokens ||
            p.flush_k->first_tile != p.plan.tiles_a - 1 || p.flush_v->first_token != (p.plan.tiles_a - 1) * kTileTokens)
            return hipErrorInvalidValue;
        p.plan.tiles_a -= 1;
    } else if (!p.seq_state && p.two_launches > 0 && p.n_kq == p.n_vq && p.plan.tiles_total > p.plan.tiles_a && p.plan.tiles_a > 0) {
        // two launches: the fp16 rows (which append the new token), and the tile that leaves the window in the step
        if (p.head_groups != 1) return hipErrorInvalidValue;
        p.rows_for_tiles = 1;
        if (hipError_t e = launch_ragged_rows(p, p.plan.tiles_total - p.plan.tiles_a, nullptr, nullptr, p.flush_k ? p.batch : 0, nullptr, stream); e != hipSuccess) return e;
    } else if (p.flush_k) {
        return hipErrorInvalidValue;
    }
    hipError_t e = hipErrorNotSupported;
    with_tiles_variant(p.bits, p.rep_here, [&](auto b, auto h) {
        constexpr int B = decltype(b)::value, H = decltype(h)::value;
        const bool cs = p.kg_shift > 0;
        if (p.seq_state) e = cs ? launch_mode<B, H, kQuantisedRagged, true>(p, stream) : launch_mode<B, H, kQuantisedRagged, false>(p, stream);
        else if (flush_inside) e = launch_mode<B, H, kFlush, false>(p, stream);
        else if (p.n_kq != p.n_vq) e = cs ? launch_mode<B, H, kMixed, true>(p, stream) : launch_mode<B, H, kMixed, false>(p, stream);
        else e = cs ? launch_mode<B, H, kWhole, true>(p, stream) : launch_mode<B, H, kWhole, false>(p, stream);
    });
    return e;
}

int tiles_max_parts(int bits, int rep) {
    int n = 0;
    with_tiles_variant(bits, rep, [&](auto b, auto h) { n = max_parts_of(decltype(b)::value, decltype(h)::value); });
    return n;
}

int tiles_resident_ragged(int bits, int rep, bool large_groups) {
    int n = 0;
    with_tiles_variant(bits, rep, [&](auto b, auto h) {
        constexpr int B = decltype(b)::value, H = decltype(h)::value;
        n = large_groups ? resident_workgroups<B, H, kQuantisedRagged, true>() : resident_workgroups<B, H, kQuantisedRagged, false>();
    });
    return n;
}

}  // namespace kivi
