// Decode attention, matrix-core family, one query head per kv-head (KIVI Equation 4 and Algorithm 1 Decoding): fp16 rows and quantised tiles of a cache in ONE launch, every byte through asynchronous copies.
//
// A unit is a (batch entry, kv-head).  Its work is a list of steps: first the fp16 rows of the window, then the
// quantised tiles.  A step gives every wavefront of a workgroup one slot of its own LDS ring: PT tiles (codes, scales,
// zero-points), or the K and V rows of NT tokens -- both are NI copies of 1 KB, so the wait for the oldest slot is one vmcnt
// with a constant and rows and tiles follow each other without a border.  A workgroup takes a run of a unit's steps; with
// several per unit each leaves a part (m, l, o[128]) in the workspace and the last one merges.  Workgroups are not
// persistent: whole units need no merge, and a new one's start is hidden behind the others of its compute unit.
//
// Arithmetic (as in decode_tiles_kernel, whose comments say why the exponents are what they are): a code left in place
// inside an fp16 lane is the exact subnormal code * 4^r * 2^-24; the matrix instruction multiplies it with q_c s_c (keys) or
// p_t s_t,g (values), split into fp16 hi + remainder in two matrix columns.  With one head 14 of 16 columns would be copies
// if every lane made the eight elements of its own column.  Instead a lane makes two elements (two channels of the key
// operand; one token, two groups of the value operand) with six or seven instructions, and the columns are
// filled through LDS; the value side's columns hold the four channel groups at once, so that a tile takes one operand.
// Key operand: q_c s_c 4^-r is exact in fp32 and its remainder is magnified by 2^11, so that it keeps 22 bits also where hi is subnormal.
// (Product and remainder in fp16, two packed instructions instead of six: launches 0.5 % shorter, but an error of 1.6e-4 of the output
// instead of 4e-6 where one channel of the query is 2^16 times the others, and 1.2e-4 instead of 4e-6 with key scales of 2^-14.  All
// factors smaller by 2^11, which saves one instruction: no faster, 1.2e-4 with key scales of 2^-14.)
// Value operand the same way, p_t 4^-r in fp32.  (p_t as two fp16 numbers and products in fp16: as many instructions, but a channel group
// whose values are 2^16 times smaller than another's had an error of 6e-4 (2 bits) and 4e-3 (4 bits) of its outputs.)
// Each lane's softmax work is one token (of 32, every token in two lanes), the one whose operand it makes.
//
// PT = 2 at 2 bits: the two tiles' chains (LDS, matrix unit, LDS, matrix unit: 0.9 us alone) overlap in one wavefront.  Three
// workgroups per compute unit hold 147 KB (2 bits) or 123 KB (4 bits) of copies in flight.  (Measured against two with three slots
// each, eight or sixteen wavefronts, one tile and four slots at 2 bits: this shape within 3 % of the best everywhere.)
//
// FLUSH (G = 32): the step in which the oldest 32 tokens leave the window takes this one launch too.  The last wavefront of a unit's
// last workgroup quantises them out of the rings into the cache and into its own slot and attends to them there; the
// others have the first items of rows and tiles to themselves meanwhile (kFlushLead).  The shares are fixed, so that a step repeats
// itself bit by bit; with a counter that hands out items the order of the sums hung on timing (11 of 11 repetitions differed at 512
// units).  Items follow each other without rounding to steps.  Counter -> fixed shares: 32 units x 4095 tokens 11.3 -> 10.7 us, 256
// x 1023 13.7 -> 12.8, 512 x 1023 19.0 -> 18.4, 512 x 4095 41.8 -> 42.6, 2048 x 2175 99.6 -> 101.5; 4 bits 128 x 2047 16.2 -> 15.1, 320 x 8191
// 77.5 -> 77.9.  (A fifth wavefront: two workgroups per compute unit instead of three.  Keys and values by a wavefront
// each, whose items go to the others: faster where compute units are idle, 128 units x 1023 tokens 11.8 -> 11.2 us, but 256 units 13.0 ->
// 13.7, 2048 units 67.0 -> 68.3.  The flushing wavefront's first item asked for before the flush: no change.)  Against a launch of its own before the attention: 8 units x 511 tokens 10.8 -> 9.6 us, 256 x 4095
// 28.1 -> 23.5, 512 x 4095 45.9 -> 41.4, 2048 x 2175 105.7 -> 103.1; 4 bits, 256 x 4095 36.4 -> 32.5, 320 x 8191 78.6 -> 77.7.  (With
// 4 bits, 800 units and more and 2000 tokens and more, steps that flush are up to 3 % longer than decode_mfma_kernel's two launches.)
//
// UNEVEN (n_kq >= n_vq, Algorithm 1's policy): the tokens between have quantised keys and fp16 value rows.  An item of those is
// MT tokens: their key tile's codes, scales and zero-points and their value rows fill a slot with the same NI copies (the key tile is
// read for every MT of its 32 tokens, from the L2 after the first); its logits go through LDS to the lanes that have the rows.  Values
// that are not there in the last tile count as scale 0.  The value token that a step quantises lies in the first of these items;
// its wavefront encodes the row that it has in LDS (a launch of its own before the attention took 4.7 us).  Items follow each
// other without rounding to steps.  Whole steps, G = 64, decode_mfma_kernel -> this one: 256 units x 4000 tokens 34.0 -> 22.7 us;
// 32 x 500 13.9 -> 8.1, 256 x 1000 26.3 -> 12.5, 512 x 4000 48.3 -> 40.0, 2048 x 2000 114.9 -> 82.7; 4 bits 32 x 500 14.7 -> 8.3, 256 x 1000
// 29.1 -> 14.8, 512 x 4000 67.4 -> 54.8, 2048 x 2000 134.8 -> 113.5; a window of 512 tokens, 256 x 4000 38.6 -> 28.0.
//
// RAGGED (sequences of different lengths, K and V split alike): a workgroup looks up its sequence -- sixty-four candidates a step -- in a table that
// the launch before made (launch_ragged_one_head, which also quantises what leaves the windows); sequences go by length, the
// longest first, and the workgroups of a unit by one_head_ragged_parts.  Whole steps, residual_rows_kernel and decode_mfma_kernel's forms for
// such batches -> this: 16 x 32 heads, 500-8000 tokens 81.4 -> 52.3 us, 4 bits 99.4 -> 73.5; 64 x 32, 500-2000 94.0 -> 70.5, 1900-2200 112.8 ->
// 93.1; 4 x 32, 100-1000 18.2 -> 14.1; 128 x 4, 50-16 000 124.6 -> 93; G = 64, 16 x 32, 500-8000 (run by run before) 160 -> 48.
//
// Bound: HBM.  A launch that only copies what this one reads takes 29.7 us for 512 units of 124 tiles at 2 bits (6.6 TB/s), rows and
// all 35; this kernel 39.4 (decode_mfma_kernel 45.5).  From 1000 to 8000 tokens at 512 units a token more costs what its bytes take at 6.1 TB/s
// (4 bits 6.6); beyond that a step has 2.5 us.  Whole steps, 2 bits, decode_mfma_kernel -> this one: 32 units x 3000 tokens 12.6 -> 9.1 us,
// 128 x 4000 22.4 -> 15.6, 256 x 1000 22.6 -> 11.3, 256 x 4000 30.0 -> 23.1, 512 x 1000 22.3 -> 15.1, 512 x 4000 45.5 -> 39.4, 768 x 4000 67.4 ->
// 56.9, 2048 x 2000 98.7 -> 87.3; 4 bits: 256 x 4000 38.6 -> 30.7, 320 x 8000 74.6 -> 72.0, 1024 x 4000 112.4 -> 111.6.
// Error against 64 bits: 7e-7 to 2e-6 of the output on plain normal data, 4e-6 to 1.6e-5 with key channels of large magnitude
// (decode_mfma_kernel 2e-5 to 2.5e-4).
#include "kivi_internal.h"
#include "kivi_quantize_tile.h"
#include "kivi_tiles_plan.h"

#include <hip/hip_fp16.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace kivi {
namespace {

using tile::half2v;
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

union Frag {            // one lane's share of a 16x16x32 fp16 operand: eight halves
    half8 h;
    half2v p[4];
    uint32_t r[4];
};

constexpr float kKeyUnscale = 4194304.0f;      // 2^22: key codes enter as code * 4^r * 2^-22
// value codes enter as code * 2^-18, times 4 in registers 1 and 3 (2 bits), or as code * 2^-22, times 16 there (4 bits)
template <int BITS> constexpr float kValueUnscale = BITS == 2 ? 262144.0f : 4194304.0f;
template <int BITS> constexpr float kValueFactor = BITS == 2 ? 4.f : 16.f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kSlack = 4;                      // log2 headroom of the running softmax reference
constexpr int kQueryExp = 8;                   // largest |q'| lies in [2^8, 2^9)
constexpr uint32_t kKeyScaleLimit = 0x54005400u;       // two times fp16 64.0
constexpr int kKeyScaleShift = 9;              // a slot with larger scales whose products pass kProductLimit takes q' 2^-9
constexpr float kProductLimit = 32768.f;
// Value side: p' = p 2^kProbExp, scales taken as s 2^-ks with s 2^-ks < 2^kValueTop; larger ones as they are while their
// products with p' stay below kValueProductLimit; ks falls back when a slot's scales are 2^-kValueWindow of that
template <int BITS> constexpr int kProbExp = BITS == 2 ? 8 : 11;
template <int BITS> constexpr int kValueTop = BITS == 2 ? 3 : 0;
constexpr int kValueWindow = 7;
constexpr float kValueProductLimit = 2048.f;

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppRor4 = 0x124, kDppRor8 = 0x128, kDppRor12 = 0x12C;

// sum / maximum over the lanes that differ in bits 4 and 5
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
__device__ __forceinline__ float row_sum(float x) {
    x += dpp<kDppXor1>(x);
    x += dpp<kDppXor2>(x);
    x += dpp<kDppHalfMirror>(x);
    return x + dpp<kDppRor8>(x);
}
__device__ __forceinline__ float wave_sum(float x) { return add_rows(row_sum(x)); }
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp<kDppXor1>(x));
    x = fmaxf(x, dpp<kDppXor2>(x));
    x = fmaxf(x, dpp<kDppHalfMirror>(x));
    return max_rows(fmaxf(x, dpp<kDppRor8>(x)));
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
__device__ __forceinline__ float2 device_load(const float* p) {
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Asynchronous copy of 16 bytes per lane: lane l's bytes land at LDS offset lds + 16 l.  (From inline asm: the compiler would
// make every LDS read wait for all copies in flight; they have no output registers, and further vector-memory
// operations only make the explicit waits stricter.  The instruction needs five wait states after a vector instruction has
// written its scalar operand, a readlane out of a spill say; the compiler does not look into the block for that.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void copy_to_lds(const void* base, uint32_t lane_offset, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(lane_offset), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void copy_to_lds(const void* lane_ptr, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds), "v"(lane_ptr) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_copies() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Products of two fp16 numbers with fp32 ones as x = hi + lo 2^-11: hi = fp16(x), and lo = fp16((x - hi) 2^11) keeps 11 bits more at any
// magnitude of x.  a, b: the fp32 factors, a_up, b_up: 2^11 times those.
constexpr float kLoMagnify = 2048.f, kLoShrink = 1.f / 2048.f;
__device__ __forceinline__ void split_products(half2v s, float a, float b, float a_up, float b_up, half2v& hi, half2v& lo) {
    // (fused operations with a zero, or with fp16 results: one mixed-precision instruction each)
    hi = half2v{(_Float16)fmaf((float)s[0], a, 0.f), (_Float16)fmaf((float)s[1], b, 0.f)};
    asm("" : "+v"(hi));                              // (or its upper half is made twice)
    lo = half2v{(_Float16)fmaf((float)hi[0], -kLoMagnify, fmaf((float)s[0], a_up, 0.f)),
                (_Float16)fmaf((float)hi[1], -kLoMagnify, fmaf((float)s[1], b_up, 0.f))};
}
__device__ __forceinline__ half2v half2_of(uint32_t x) { return __builtin_bit_cast(half2v, x); }

// Code fragments of tile coordinate u = 2 pair + odd: codes as high in the mantissa as they go (keys at bits 2, 4, 6, 8 or 2, 6;
// values at 6, 8 or 2, 6), see decode_tiles_kernel.  (4-bit values all at bit 6: 64 instead of 48 instructions a tile, launches 1 %
// longer, error 2.5e-6 instead of 1.2e-5 of the output; 2-bit values at 2, 4, 6, 8: no faster, 4e-5 instead of 7e-6.)
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
        return key_fragment<BITS>(w, pair, odd);
    }
    return f.h;
}

template <int BITS, int PT, int NB, int WV>
struct Shape {
    static constexpr int kCodeBytes = kTileTokens * kHeadDim * BITS / 8;
    static constexpr int kTileBytes = 2 * kCodeBytes + 1024;
    static constexpr int kSlotBytes = PT * kTileBytes;
    static constexpr int kPlanes = BITS / 2;
    static constexpr int NI = PT * (2 * kPlanes + 1);          // copy instructions per slot
    static constexpr int NT = 2 * NI;                          // tokens whose fp16 rows (K and V) fill a slot
    // what a flush weighs as a part's work: a step at 2 bits, two of half the tiles at 4 (320 units x 8191, 4 bits: 78.7 us with
    // one, 77.0 with two or three; 32 x 8191 at 2 bits: 24.4, 24.6, 25.2 us with one, two, three)
    static constexpr int kFlushSteps = 2 / PT;
    // Items that each other wavefront of its workgroup takes before the flushing one takes its first: where all workgroups run at
    // once, and where there are more than fit (the others of a compute unit use the time of a flush then).  2 bits, 256 units x 1023
    // tokens 13.9 / 12.8 / 12.2 us with 4 / 5 / 6, 512 x 4095 43.2 / 42.6 / 43.1; 2048 x 1023 66.4 / 65.9 / 66.4 with 1 / 2 / 5; 4 bits, 256 x 4095 34.1 /
    // 33.7 with 5 / 6, 320 x 8191 77.5 / 77.5 / 78.9 with 6 / 8 / 16.
    static constexpr int kFlushLead = PT == 2 ? 5 : 6, kFlushLeadMany = PT == 2 ? 2 : 3;
    // a slot of a key tile's codes, its scales and zero-points, and MT tokens' fp16 value rows
    static constexpr int MT = 4 * (NI - kPlanes - 1), kMixedRows = kCodeBytes + 1024;
    // operands of a tile: key side hi (128 halves), 16 halves of skew, lo; value side 8 columns of 32 tokens
    static constexpr int kKeyColumn = 144, kOperandHalves = 272;
    static constexpr int kWaveBytes = NB * kSlotBytes + PT * kOperandHalves * 2;
    static constexpr int kLds = WV * kWaveBytes + WV * 8 + 16;
};

// The sequence of workgroup wg: the last whose first workgroup is not after it.  Sixty-four candidates at a time.
__device__ __forceinline__ OneHeadSequence find_sequence(const DecodeParams& p, int wg, int lane) {
    int lo = 0, n = p.batch;                           // among [lo, lo + n)
    while (n > 1) {
        const int stride = (n + 63) / 64, i = lane * stride;
        const bool not_after = i < n && p.unit_parts[lo + i] <= wg;
        const int at = (__popcll(__builtin_amdgcn_ballot_w64(not_after)) - 1) * stride;
        lo += at;
        n = min(stride, n - at);
    }
    // (through the scalar cache)
    const auto* e = reinterpret_cast<const __attribute__((address_space(4))) int32_t*>(reinterpret_cast<uintptr_t>(p.wave_desc)) + 8 * lo;
    return OneHeadSequence{e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7]};
}

// RAGGED: sequences of different lengths.
template <int BITS, int PT, int NB, int WV, int OCC, bool CS, bool FLUSH, bool UNEVEN, bool RAGGED>
__global__ __launch_bounds__(64 * WV, OCC * WV / 4) void decode_one_kernel(DecodeParams p) {
    using S = Shape<BITS, PT, NB, WV>;
    static_assert(!(CS && FLUSH), "a flush in this launch: G = 32");
    static_assert(!(UNEVEN && FLUSH), "K and V split differently: a flush of one value token only");
    static_assert(!(RAGGED && (UNEVEN || FLUSH)), "different lengths: K and V split alike, flushed before");
    constexpr int NI = S::NI, NT = S::NT, NR = (NT + 3) / 4, MT = S::MT;
    __shared__ __align__(16) unsigned char sm[S::kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kb = lane >> 4;
    const bool is_lo = n >= 8;
    const int kg = CS ? p.kg_shift : 0;
    unsigned char* ring = sm + wave * S::kWaveBytes;
    unsigned char* sm_query = ring + NB * S::kSlotBytes;                        // (until the first operands are made)
    _Float16* operand = reinterpret_cast<_Float16*>(sm_query);
    float (*sm_ml)[2] = reinterpret_cast<float (*)[2]>(sm + WV * S::kWaveBytes);
    int& sm_last = *reinterpret_cast<int*>(sm + WV * S::kWaveBytes + WV * 8);
    const uint32_t ring_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)ring);

    // ---- this workgroup's run of its unit's steps ----
    int u, part;
    if constexpr (RAGGED) {
        const OneHeadSequence s = find_sequence(p, blockIdx.x, lane);
        const int at = (int)blockIdx.x - s.first_wg, head = at / s.parts;
        u = s.sequence * p.n_kv_heads + head;
        part = at - head * s.parts;
        p.n_kq = p.n_vq = s.n_q;
        p.n_kr = p.n_vr = s.n_r;
        p.k_r_start = s.k_start;
        p.v_r_start = s.v_start;
        p.plan.tiles_a = s.n_q / kTileTokens;
        p.unit_wgs = s.parts;
        p.axis_len = s.steps / s.parts;
        p.axis_rem = s.steps - p.axis_len * s.parts;
    } else {
        u = blockIdx.x / p.unit_wgs;
        part = blockIdx.x % p.unit_wgs;
    }
    const int n_kr = p.n_kr;
    // UNEVEN: tokens below v_q have quantised values in the cache, the others rows in the ring from slot v_start on
    const int v_q = p.n_vq - p.flushed_values;
    const int v_start = !UNEVEN || p.v_r_start >= p.flushed_values ? p.v_r_start - (UNEVEN ? p.flushed_values : 0) : p.cap_r - 1;
    const int v_skip = UNEVEN ? p.n_kq - v_q : 0;                                // value rows before the window's
    const int tiles = UNEVEN ? (v_q + kTileTokens - 1) / kTileTokens : p.plan.tiles_a - FLUSH;      // (the flushed tile is the last)
    using Work = OneHeadItems<BITS, FLUSH, UNEVEN>;
    static_assert(std::is_same_v<Work, OneHeadWork<WV, PT, S::NT, S::MT, S::kFlushSteps, FLUSH, UNEVEN>>);
    Work work(StepAxis{p.axis_len, p.axis_rem}, part, p.unit_wgs, tiles, p.n_kq, v_q, n_kr);
    // the last wavefront of a unit's last workgroup quantises the tokens that leave the window before it takes its share
    const bool flushes = FLUSH && part == p.unit_wgs - 1 && wave == WV - 1;
    const int n_items = work.n_items, n_row_items = work.n_row_items, n_fp16_items = work.n_fp16_items;
    const int64_t unit = u;

    // ---- copies ----
    const uint32_t lane16 = lane * 16;
    const int64_t tile0 = unit * p.cap_tiles;
    // lanes 0-15 k_scale, 16-31 k_zero, 32-47 v_scale, 48-63 v_zero
    const char* sc = reinterpret_cast<const char*>(kb == 0 ? p.k_scale : kb == 1 ? p.k_zero : kb == 2 ? p.v_scale : p.v_zero);
    sc += CS && kb >= 2 ? min(n * 16, (256 >> kg) - 16) : n * 16;
    auto copy_tiles = [&](int t0, int slot) {
        const uint32_t dst = ring_lds + slot * S::kSlotBytes;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");             // the slot's last readers have their data
#pragma unroll
        for (int t = 0; t < PT; ++t) {
            const int64_t tile = tile0 + min(t0 + t, tiles - 1);
            const char* kc = reinterpret_cast<const char*>(p.k_codes) + tile * S::kCodeBytes;
            const char* vc = reinterpret_cast<const char*>(p.v_codes) + tile * S::kCodeBytes;
#pragma unroll
            for (int pl = 0; pl < S::kPlanes; ++pl) {
                copy_to_lds(kc + pl * 1024, lane16, dst + t * S::kTileBytes + pl * 1024);
                copy_to_lds(vc + pl * 1024, lane16, dst + t * S::kTileBytes + S::kCodeBytes + pl * 1024);
            }
            int64_t off = tile * 256;
            if constexpr (CS) off = kb < 2 ? (tile >> kg) * 256 : (tile * 256) >> kg;
            copy_to_lds(sc + off, dst + t * S::kTileBytes + 2 * S::kCodeBytes);
        }
    };
    // key rows of the window's tokens t0 .. t0 + NT - 1, then value rows, 256 bytes each (past the end the last token's again;
    // the newest token's out of k_new / v_new)
    auto copy_rows = [&](int t0, int slot) {
        const uint32_t dst = ring_lds + slot * S::kSlotBytes;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int r = 4 * j + kb;
            const bool is_v = r >= NT;
            const int t = min(t0 + (is_v ? r - NT : r), n_kr - 1);
            const __half* src = (is_v ? p.v_resid : p.k_resid) + (unit * p.cap_r + ring_slot(is_v ? v_start : p.k_r_start, is_v ? t + v_skip : t, p.cap_r)) * kHeadDim;
            if (p.k_new && t == n_kr - 1) src = (is_v ? p.v_new : p.k_new) + unit * kHeadDim;
            copy_to_lds(src + n * 8, dst + j * 1024);
        }
    };
    // tokens t0 .. t0 + MT - 1 of a key tile, and their value rows (before the first: that one's again)
    auto copy_mixed = [&](int t0, int slot) {
        const uint32_t dst = ring_lds + slot * S::kSlotBytes;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int64_t tile = tile0 + t0 / kTileTokens;
        const char* kc = reinterpret_cast<const char*>(p.k_codes) + tile * S::kCodeBytes;
#pragma unroll
        for (int pl = 0; pl < S::kPlanes; ++pl) copy_to_lds(kc + pl * 1024, lane16, dst + pl * 1024);
        int64_t off = tile * 256;
        if constexpr (CS) off = kb < 2 ? (tile >> kg) * 256 : (tile * 256) >> kg;
        copy_to_lds(sc + off, dst + S::kCodeBytes);
#pragma unroll
        for (int j = 0; j < MT / 4; ++j)
            copy_to_lds(p.v_resid + (unit * p.cap_r + ring_slot(v_start, max(t0 + 4 * j + kb - v_q, 0), p.cap_r)) * kHeadDim + n * 8, dst + S::kMixedRows + j * 1024);
    };
    // the query
    if (lane < 16) copy_to_lds(p.q + unit * kHeadDim + n * 8, (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)sm_query));
    work.order(part, p.unit_wgs, u, p.one_round ? S::kFlushLead : S::kFlushLeadMany);
    auto copy_item = [&](int item, int slot) {
        if (item < n_row_items) copy_rows(work.row_of(item), slot);
        else if (UNEVEN && item < n_fp16_items) copy_mixed(work.mixed_of(item), slot);
        else if (item < n_items) copy_tiles(work.tile_of(item), slot);
    };
    int now = flushes ? n_items : work.first(wave, false), next = work.after(now);
    copy_item(now, 0);
    copy_item(next, 1);

    // ---- the tokens that leave the window in this step: quantised out of the rings into the cache and into this
    // wavefront's slot, where it attends to them like to any tile ----
    if constexpr (FLUSH) {
        if (flushes) {
            __builtin_amdgcn_s_setprio(3);             // (the longest chain of a short launch)
            tile::flush_tile<BITS>(p, unit, tile0 + tiles, lane, ring, true);
            wave_lds_sync();
        }
    }

    // ---- state ----
    // own_tok, own_pair: the token (of every tile) and the channel groups 2 own_pair, + 1 whose value operand this lane makes
    const int own_i = (n >> 1) & 3, own_pair = n & 1, own_tok = kb * 4 + own_i + (is_lo ? 16 : 0);
    const float own_exp = own_i & 2 ? (BITS == 2 ? 2.f : 4.f) : 0.f;       // log2 of that token's code position factor
    const int my_group = (n & 1) * 2 + ((n >> 1) & 1);
    float4v acc[8];
    // acc[u][i]: value code sums of channel 16 u + 4 kb + i, column n (of use where its group is u >> 1); z_own: zero-point sums of
    // this lane's tokens and groups; r_out: the fp16 rows' outputs of channels 8 n .. over rows kb, kb + 4, ..; mref: reference
    // (log2) of the probabilities, l_lane, r_l: sums of this lane's
    float z_own[2] = {0.f, 0.f}, r_out[8], r_l = 0.f, l_lane = 0.f, mref = -INFINITY;
#pragma unroll
    for (int u8 = 0; u8 < 8; ++u8) acc[u8] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < 8; ++e) r_out[e] = 0.f;
    int ks = 0;
    bool ks_set = false;
    uint32_t value_limit = 0;

    // the query has arrived, the first slots are on their way
    if (next < n_items) wait_copies<2 * NI>();
    else if (now < n_items) wait_copies<NI>();
    else if (!flushes) wait_copies<0>();               // (the rows of a flush have come after the query)
    asm volatile("" ::: "memory");
    // c_own, c_other: factors of the key products of this lane's column and of its partner's (hi and lo, or lo and hi);
    // qk, qk_up: this lane's two channels of q' over the codes' position factors, and 2^11 times those
    float c_own, c_other, c_zero, qk[2], qk_up[2];
    half2v q_own;
    const half8 q_row = *reinterpret_cast<const half8*>(sm_query + n * 16);
    {
        const half2v raw = *reinterpret_cast<const half2v*>(sm_query + lane * 4);
        const float mx = wave_max(fmaxf(fabsf((float)raw[0]), fabsf((float)raw[1])));
        const bool on = mx > 0.f;
        const int a = on ? min(kQueryExp + 127 - (int)(__float_as_uint(mx) >> 23), 28) : 0;
        c_zero = p.softmax_scale * kLog2e;
        const float c_code = c_zero * kKeyUnscale * __uint_as_float((uint32_t)(127 - a) << 23);
        c_own = is_lo ? c_code * kLoShrink : c_code;
        c_other = is_lo ? c_code : c_code * kLoShrink;
        q_own = raw;                                   // (zero-points meet the query as it is: exact products, sums in fp32)
        const float f = on ? __uint_as_float((uint32_t)(127 + a - (BITS == 2 ? 2 * (lane & 3) : 4 * (lane & 1))) << 23) : 0.f;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            qk[i] = (float)raw[i] * f;
            qk_up[i] = qk[i] * kLoMagnify;
        }
    }

    auto rescale = [&](float f) {
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8) acc[u8] *= f;
        z_own[0] *= f;
        z_own[1] *= f;
#pragma unroll
        for (int e = 0; e < 8; ++e) r_out[e] *= f;
        r_l *= f;
        l_lane *= f;
    };
    auto raise_reference = [&](float top) {                                 // top: a lane's largest logit
        const float mnew = fmaxf(mref, wave_max(top));
        rescale(mref == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mref - mnew));
        mref = mnew;
    };
    auto max_pairs = [&](uint32_t a, uint32_t b) -> uint32_t {              // non-negative fp16 compare as integers
        typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2v, a), __builtin_bit_cast(ushort2v, b)));
    };
    auto any_above = [&](uint32_t s2, uint32_t limit) -> bool { return __any(max_pairs(s2, limit) != limit); };
    auto top_scale = [&](int k) -> uint32_t {
        const int top = k + kValueTop<BITS> + 15;                           // biased fp16 exponent
        const uint32_t lim = top >= 31 ? 0x7BFFu : top <= 0 ? 0u : (uint32_t)(top << 10) - 1;
        return lim | lim << 16;
    };
    auto fit_value_exponent = [&](uint32_t s2, auto&& top_product) {
        if (!any_above(s2, value_limit)) return;
        bool high = true;
        if (ks > 0) {
            high = any_above(s2, top_scale(ks));
            if (!high && any_above(s2, (uint32_t)(ks + kValueTop<BITS> - kValueWindow + 15) * 0x04000400u)) return;
        }
        const float mx = wave_max(fmaxf((float)half2_of(s2)[0], (float)half2_of(s2)[1]));
        const int want = __builtin_amdgcn_readfirstlane(max((int)(__float_as_uint(mx) >> 23) - 126 - kValueTop<BITS>, -24));
        int next = max(want, 0);
        if (high) {
            next = ks_set && ks >= 0 ? ks : want > -kValueWindow ? 0 : want;
            if (want > next && __any(top_product() > kValueProductLimit * __uint_as_float((uint32_t)(127 + next) << 23))) next = want;
        }
        if (ks_set) {
            const float f = __uint_as_float((uint32_t)(127 + ks - next) << 23);
#pragma unroll
            for (int u8 = 0; u8 < 8; ++u8) acc[u8] *= f;
        }
        ks = next;
        ks_set = true;
        value_limit = ks > 0 ? 0 : top_scale(ks);
    };
    auto own_of = [&](const float4v& x) -> float {
        const float a = own_i & 1 ? x[1] : x[0], b = own_i & 1 ? x[3] : x[2];
        return own_i & 2 ? b : a;
    };

    auto load_codes = [&](const unsigned char* at, uint32_t (&w)[2 * BITS]) {
#pragma unroll
        for (int pl = 0; pl < S::kPlanes; ++pl) {
            const uint4v v = *reinterpret_cast<const uint4v*>(at + pl * 1024 + lane16);
            w[4 * pl + 0] = v[0]; w[4 * pl + 1] = v[1]; w[4 * pl + 2] = v[2]; w[4 * pl + 3] = v[3];
        }
    };
    const int value_at = CS ? own_tok * (8 >> kg) + ((2 * own_pair) >> kg) * 2 : own_tok * 8 + own_pair * 4;
    auto value_pair = [&](const unsigned char* at) -> uint32_t {
        if constexpr (CS) {
            const uint32_t h = *reinterpret_cast<const uint16_t*>(at + value_at);
            return h | h << 16;
        } else {
            return *reinterpret_cast<const uint32_t*>(at + value_at);
        }
    };
    // logits (log2) of this lane's token of N tiles; s_raw: their scales, top: the largest
    auto logits = [&](auto count, const auto& kw, const auto& s_raw, const auto& z, uint32_t top, auto& x) {
        constexpr int N = decltype(count)::value;
        auto put_operands = [&](const uint32_t (&sr)[N], float f) {
#pragma unroll
            for (int t = 0; t < N; ++t) {
                half2v hi, lo;
                split_products(half2_of(sr[t]), qk[0] * f, qk[1] * f, qk_up[0] * f, qk_up[1] * f, hi, lo);
                _Float16* b = operand + t * S::kOperandHalves;
                *reinterpret_cast<half2v*>(b + 2 * lane) = hi;
                *reinterpret_cast<half2v*>(b + S::kKeyColumn + 2 * lane) = lo;
            }
        };
        float f_own = c_own, f_other = c_other;
        bool shift = false;
        if (any_above(top, kKeyScaleLimit)) {          // (rare, and kept apart: nothing of it is to move into the ordinary path)
            uint32_t sr[N];
            float a = 0.f;
#pragma unroll
            for (int t = 0; t < N; ++t) {
                asm("" : "=v"(sr[t]) : "0"(s_raw[t]));
                a = fmaxf(a, fmaxf(fabsf(qk[0] * (float)half2_of(sr[t])[0]), fabsf(qk[1] * (float)half2_of(sr[t])[1])));
            }
            shift = __any(a > kProductLimit);
            if (shift) {
                put_operands(sr, 1.f / (1 << kKeyScaleShift));
                f_own *= (float)(1 << kKeyScaleShift);
                f_other *= (float)(1 << kKeyScaleShift);
                asm volatile("" ::: "memory");
            }
        }
        if (!shift) put_operands(s_raw, 1.f);
        wave_lds_sync();
        half8 f[N][4];
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
                f[t][cb] = *reinterpret_cast<const half8*>(operand + t * S::kOperandHalves + (is_lo ? S::kKeyColumn : 0) + cb * 32 + kb * 8);
        float zk[N];
#pragma unroll
        for (int t = 0; t < N; ++t) zk[t] = wave_sum(__builtin_amdgcn_fdot2(q_own, z[t], 0.f, false)) * c_zero;
        float4v d[N][2];
#pragma unroll
        for (int t = 0; t < N; ++t) d[t][0] = d[t][1] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int t = 0; t < N; ++t) {
                d[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(key_fragment<BITS>(kw[t], cb, 0), f[t][cb], d[t][0], 0, 0, 0);
                d[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(key_fragment<BITS>(kw[t], cb, 1), f[t][cb], d[t][1], 0, 0, 0);
            }
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const float x0 = own_of(d[t][0]), x1 = own_of(d[t][1]);
            x[t] = fmaf(is_lo ? x1 : x0, f_own, fmaf(dpp<kDppRor8>(is_lo ? x0 : x1), f_other, zk[t]));
        }
    };
    // N tiles of a slot; live: those that are there (UNEVEN: tokens that are there)
    auto quantised = [&](auto count, const unsigned char* sl, int live) {
        constexpr int N = decltype(count)::value;
        constexpr int kS = 2 * S::kCodeBytes;
        auto there = [&](int t) -> bool { return UNEVEN ? t * kTileTokens + own_tok < live : t == 0 || t < live; };
        uint32_t kw[N][2 * BITS], vw[N][2 * BITS], s_raw[N], v_raw[N], top = 0;
        half2v z[N], vz[N];
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const unsigned char* at = sl + t * S::kTileBytes;
            s_raw[t] = *reinterpret_cast<const uint32_t*>(at + kS + lane * 4);
            z[t] = half2_of(*reinterpret_cast<const uint32_t*>(at + kS + 256 + lane * 4));
            load_codes(at, kw[t]);
            v_raw[t] = value_pair(at + kS + 512);
            vz[t] = half2_of(value_pair(at + kS + 768));
            load_codes(at + S::kCodeBytes, vw[t]);
            if (UNEVEN && !there(t)) {                 // (never written)
                v_raw[t] = 0;
                vz[t] = half2v{0, 0};
            }
            top = max_pairs(top, s_raw[t]);
        }
        float x[N], pv[N], mx = -INFINITY;
        logits(count, kw, s_raw, z, top, x);
        // this lane's token of every tile: probability over the code's position factor
#pragma unroll
        for (int t = 0; t < N; ++t) {
            if (!there(t)) x[t] = -INFINITY;
            mx = fmaxf(mx, x[t]);
        }
        if (__any(mx > mref + (float)kSlack)) raise_reference(mx);
        const float off = (float)kProbExp<BITS> - own_exp - mref;
        uint32_t vtop = 0;
#pragma unroll
        for (int t = 0; t < N; ++t) {
            pv[t] = __builtin_amdgcn_exp2f(x[t] + off);
            l_lane += pv[t];
            if (UNEVEN || there(t)) vtop = max_pairs(vtop, v_raw[t]);
        }
        fit_value_exponent(vtop, [&]() {
            float m = 0.f;
#pragma unroll
            for (int t = 0; t < N; ++t) m = fmaxf(m, pv[t] * fmaxf((float)half2_of(v_raw[t])[0], (float)half2_of(v_raw[t])[1]));
            return m;
        });
        const float pk = __uint_as_float((uint32_t)(127 - ks) << 23), pk_up = pk * kLoMagnify;
#pragma unroll
        for (int t = 0; t < N; ++t) {
            half2v hi, lo;
            const float ps = pv[t] * pk, ps_up = pv[t] * pk_up;
            split_products(half2_of(v_raw[t]), ps, ps, ps_up, ps_up, hi, lo);
            z_own[0] = fmaf(pv[t], (float)vz[t][0], z_own[0]);
            z_own[1] = fmaf(pv[t], (float)vz[t][1], z_own[1]);
            _Float16* col = operand + t * S::kOperandHalves + own_pair * 4 * 32 + own_tok;         // columns (group, hi / lo)
            col[0] = hi[0];
            col[32] = lo[0];
            col[64] = hi[1];
            col[96] = lo[1];
        }
        wave_lds_sync();
        half8 fv[N];
#pragma unroll
        for (int t = 0; t < N; ++t)
            fv[t] = *reinterpret_cast<const half8*>(operand + t * S::kOperandHalves + (my_group * 2 + (is_lo ? 1 : 0)) * 32 + kb * 8);
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int u8 = 0; u8 < 8; ++u8)
                acc[u8] = __builtin_amdgcn_mfma_f32_16x16x32_f16(value_fragment<BITS>(vw[t], u8 >> 1, u8 & 1), fv[t], acc[u8], 0, 0, 0);
        wave_lds_sync();
    };
    // NT tokens' fp16 rows; lane (n, kb) takes channels 8 n .. of rows kb, kb + 4, ..
    auto fp16_rows = [&](const unsigned char* sl, int left) {
        const float c_row = p.softmax_scale * kLog2e;
        float x[NR], mx = -INFINITY;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            Frag k, q;
            k.h = *reinterpret_cast<const half8*>(sl + (4 * j + kb) * 256 + n * 16);
            q.h = q_row;
            float a = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) a = __builtin_amdgcn_fdot2(k.p[r], q.p[r], a, false);
            x[j] = 4 * j + kb < min(left, NT) ? row_sum(a) * c_row : -INFINITY;
            mx = fmaxf(mx, x[j]);
        }
        if (__any(mx > mref + (float)kSlack)) raise_reference(mx);
        const float ref = RAGGED && mref == -INFINITY ? 0.f : mref;              // (every logit so far is -inf: they count for nothing)
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            const float pr = __builtin_amdgcn_exp2f(x[j] + ((float)kProbExp<BITS> - ref));
            r_l += pr;
            const half8 v = *reinterpret_cast<const half8*>(sl + NT * 256 + min(4 * j + kb, NT - 1) * 256 + n * 16);
#pragma unroll
            for (int e = 0; e < 8; ++e) r_out[e] = fmaf(pr, (float)v[e], r_out[e]);
        }
        if (p.k_new && left <= NT && kb < 2) {                                    // the newest token's rows go to the rings
            const uint4v row = *reinterpret_cast<const uint4v*>(sl + (kb * NT + left - 1) * 256 + n * 16);
            const int at = ring_slot(kb ? v_start : p.k_r_start, kb ? n_kr - 1 + v_skip : n_kr - 1, p.cap_r);
            *reinterpret_cast<uint4v*>(const_cast<__half*>(kb ? p.v_resid : p.k_resid) + (unit * p.cap_r + at) * kHeadDim + n * 8) = row;
        }
    };
    // The value token that is quantised in this step, its row in LDS: codes and group constants to the cache, the row
    // becomes its codes.  A lane has channels 32 j + i and 16 on, j = lane % 4, i = lane / 4: one word of the tile, whose
    // other codes stay.  Returns scale and zero-point of this lane's channels 8 n ..
    auto flush_value = [&](_Float16* row) -> float2 {
        constexpr float levels = (float)((1 << BITS) - 1);
        const int j = lane & 3, i = lane >> 2, e = v_q & 7;
        const float a = (float)row[32 * j + i], b = (float)row[32 * j + 16 + i];
        float lo = -fminf(a, b), hi = fmaxf(a, b);
        lo = max_rows(fmaxf(fmaxf(lo, dpp<kDppRor4>(lo)), fmaxf(dpp<kDppRor8>(lo), dpp<kDppRor12>(lo))));
        hi = max_rows(fmaxf(fmaxf(hi, dpp<kDppRor4>(hi)), fmaxf(dpp<kDppRor8>(hi), dpp<kDppRor12>(hi))));
        if (kg >= 1) {
            lo = fmaxf(lo, dpp<kDppXor1>(lo));
            hi = fmaxf(hi, dpp<kDppXor1>(hi));
        }
        if (kg >= 2) {
            lo = fmaxf(lo, dpp<kDppXor2>(lo));
            hi = fmaxf(hi, dpp<kDppXor2>(hi));
        }
        const __half s16 = __float2half_rn((hi + lo) / levels);
        const float s = __half2float(s16), z = -lo;
        const uint32_t ca = tile::encode(a, z, s, levels), cb = tile::encode(b, z, s, levels);
        const int64_t at = tile0 + v_q / kTileTokens;
        const int half_word = BITS == 2 ? j : 2 * j + (e >> 2);
        uint32_t* word = const_cast<uint32_t*>(p.v_codes) + at * (S::kCodeBytes / 4) + (half_word >> 2) * 256 + ((v_q >> 3 & 3) * 16 + i) * 4 + (half_word & 3);
        const int bit = (e & 1) * 16 + (BITS == 2 ? 2 * (e >> 1) : 4 * (e >> 1 & 1));
        constexpr uint32_t mask = BITS == 2 ? 0x303u : 0xF0Fu;
        *word = (*word & ~(mask << bit)) | (ca | cb << 8) << bit;
        if (i == 0 && (j & ((1 << kg) - 1)) == 0) {
            const int64_t o = (at * kTileTokens + (v_q & (kTileTokens - 1))) * (4 >> kg) + (j >> kg);
            const_cast<__half*>(p.v_scale)[o] = s16;
            const_cast<__half*>(p.v_zero)[o] = __float2half_rn(z);
        }
        row[32 * j + i] = (_Float16)(float)ca;
        row[32 * j + 16 + i] = (_Float16)(float)cb;
        wave_lds_sync();
        return make_float2(__shfl(s, n >> 2), __shfl(z, n >> 2));
    };
    // MT tokens with quantised keys and fp16 value rows, the first is t0: one key tile's logits, the probabilities through
    // LDS to the lanes that have the rows
    auto mixed = [&](unsigned char* sl, int t0) {
        uint32_t kw[1][2 * BITS], s_raw[1];
        half2v z[1];
        float x[1];
        s_raw[0] = *reinterpret_cast<const uint32_t*>(sl + S::kCodeBytes + lane * 4);
        z[0] = half2_of(*reinterpret_cast<const uint32_t*>(sl + S::kCodeBytes + 256 + lane * 4));
        load_codes(sl, kw[0]);
        logits(std::integral_constant<int, 1>{}, kw, s_raw, z, s_raw[0], x);
        const int t = (t0 & -kTileTokens) + own_tok;
        if (t < max(t0, v_q) || t >= t0 + MT) x[0] = -INFINITY;
        if (__any(x[0] > mref + (float)kSlack)) raise_reference(x[0]);
        float* pr_of = reinterpret_cast<float*>(operand);
        wave_lds_sync();
        pr_of[own_tok] = __builtin_amdgcn_exp2f(x[0] + ((float)kProbExp<BITS> - mref));
        const int flushed = p.flushed_values && v_q >= t0 ? v_q - t0 : MT;        // (v_q is in the first of these items)
        float2 sz = {1.f, 0.f};
        if (flushed < MT) sz = flush_value(reinterpret_cast<_Float16*>(sl + S::kMixedRows + flushed * 256));
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < MT / 4; ++j) {
            const int r = 4 * j + kb;
            const float pr = pr_of[(t0 & (kTileTokens - 1)) + r];
            const bool coded = r == flushed;
            const float by = coded ? pr * sz.x : pr, plus = coded ? pr * sz.y : 0.f;
            r_l += pr;
            const half8 v = *reinterpret_cast<const half8*>(sl + S::kMixedRows + r * 256 + n * 16);
#pragma unroll
            for (int c = 0; c < 8; ++c) r_out[c] = fmaf(by, (float)v[c], r_out[c] + plus);
        }
        wave_lds_sync();
    };
    // The instruction arbiter favours the oldest wavefront of a SIMD.  Where all workgroups start at once the younger ones would
    // end late and alone (512 units: 28 against 36 us), so a wavefront's priority falls with the share of its work that is done (39.6 ->
    // 38.7 us); with more workgroups than fit at once the oldest ones' head start is what hides the others' starts (2048
    // units: 87 us as it is, 91 with falling priorities).
    const int quarter = p.one_round ? n_items >> 2 : 0x1fffffff;
    auto begin = [&]() {
        const int left = n_items - now;
        if (left > 3 * quarter) __builtin_amdgcn_s_setprio(3);
        else if (left > 2 * quarter) __builtin_amdgcn_s_setprio(2);
        else if (left > quarter) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
        if (next < n_items) wait_copies<NI>();
        else wait_copies<0>();
    };
    int slot = 0;
    auto end = [&]() {
        now = next;
        next = work.after(next);
        copy_item(next, slot);
        slot ^= 1;
    };
    if constexpr (FLUSH) {
        if (flushes) {
            quantised(std::integral_constant<int, 1>{}, ring, 1);
            now = work.first(wave, true);
            copy_item(now, 0);
            next = work.after(now);
            copy_item(next, 1);
        }
    }
#pragma unroll 1
    while (now < n_row_items) {
        begin();
        const int left = n_kr - work.row_of(now);
        if (left > 0) fp16_rows(ring + slot * S::kSlotBytes, left);
        end();
    }
    if constexpr (UNEVEN) {
#pragma unroll 1
        while (now < n_fp16_items) {
            begin();
            mixed(ring + slot * S::kSlotBytes, work.mixed_of(now));
            end();
        }
    }
#pragma unroll 1
    while (now < n_items) {
        begin();
        const int live = UNEVEN ? v_q - work.tile_of(now) * kTileTokens : tiles - work.tile_of(now);
        if (live > 0) quantised(std::integral_constant<int, PT>{}, ring + slot * S::kSlotBytes, live);
        end();
    }

    // ---- merge the wavefronts (their rings are free) ----
    float* o_wave = reinterpret_cast<float*>(ring);
    {
        const float l = wave_sum(l_lane * (own_i & 2 ? 0.5f * kValueFactor<BITS> : 0.5f) + r_l * (1.f / 16));
        if (lane == 0) {
            sm_ml[wave][0] = mref;
            sm_ml[wave][1] = l;
        }
        float zo[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float t = z_own[k] * (own_i & 2 ? kValueFactor<BITS> : 1.f);
            t += dpp<kDppXor2>(t);
            t += dpp<kDppRor4>(t);
            t += dpp<kDppRor8>(t);
            zo[k] = add_rows(t);
        }
        const float up = kValueUnscale<BITS> * __uint_as_float((uint32_t)(127 + ks) << 23);
#pragma unroll
        for (int u8 = 0; u8 < 8; ++u8) {
            float4v o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = fmaf(fmaf(dpp<kDppRor8>(acc[u8][i]), kLoShrink, acc[u8][i]), up, zo[(u8 >> 1) & 1]);     // (of use in the lanes of hi)
            if (n < 4 && my_group == u8 >> 1) *reinterpret_cast<float4v*>(&o_wave[u8 * 16 + kb * 4]) = o;
        }
        if (n_fp16_items > 0) {
            float r[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = add_rows(r_out[e]);
            wave_lds_sync();
            if (kb == 0) {
                float4v* o = reinterpret_cast<float4v*>(&o_wave[n * 8]);
                o[0] += float4v{r[0], r[1], r[2], r[3]};
                o[1] += float4v{r[4], r[5], r[6], r[7]};
            }
        }
    }
    lds_barrier();
    const int parts = p.unit_wgs;
    float m = -INFINITY, ll = 0.f;
#pragma unroll
    for (int w = 0; w < WV; ++w) m = fmaxf(m, sm_ml[w][0]);
    float2 oo = {0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WV; ++w) {
        const float mw = sm_ml[w][0];
        const float f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - m);
        const float2 x = *reinterpret_cast<const float2*>(sm + w * S::kWaveBytes + lane * 8);
        ll = fmaf(sm_ml[w][1], f, ll);
        oo.x = fmaf(x.x, f, oo.x);
        oo.y = fmaf(x.y, f, oo.y);
    }
    m -= (float)kProbExp<BITS>;
    float* out = p.out + unit * kHeadDim + 2 * lane;
    if (parts == 1) {
        if (wave == 0) *reinterpret_cast<float2*>(out) = make_float2(oo.x / ll, oo.y / ll);
        return;
    }
    const int64_t prow = unit * p.part_stride;
    if (wave == 0) {
        device_store(p.part_o + (prow + part) * kHeadDim + 2 * lane, oo);
        if (lane == 0) device_store(p.part_ml + (prow + part) * 2, make_float2(m, ll));
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) {
            const int done = __hip_atomic_fetch_add(p.counters + u, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sm_last = done == parts - 1;
        }
    }
    lds_barrier();
    if (!sm_last) return;
    // ---- the last workgroup merges: wavefront w takes parts w, w + 4, ..; lane: two channels ----
    {
        constexpr int kBatch = 8;
        const float* po = p.part_o + prow * kHeadDim + 2 * lane;
        float2 ov[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) ov[j] = device_load(po + (int64_t)min(wave + WV * j, parts - 1) * kHeadDim);
        float2 st[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) st[k] = device_load(p.part_ml + (prow + min(lane + 64 * k, parts - 1)) * 2);
        const float mm = wave_max(fmaxf(st[0].x, st[1].x));
        float wt[2], lsum = 0.f;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            wt[k] = lane + 64 * k < parts && st[k].x != -INFINITY ? __builtin_amdgcn_exp2f(st[k].x - mm) : 0.f;
            lsum = fmaf(st[k].y, wt[k], lsum);
        }
        lsum = wave_sum(lsum);
        float2 o = {0.f, 0.f};
        for (int i0 = 0; wave + i0 < parts; i0 += WV * kBatch) {
            if (i0 > 0) {
#pragma unroll
                for (int j = 0; j < kBatch; ++j) ov[j] = device_load(po + (int64_t)min(wave + i0 + WV * j, parts - 1) * kHeadDim);
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int i = wave + i0 + WV * j;                                // (weights are 0 past the last part)
                const float w = __int_as_float(i < 64 ? __builtin_amdgcn_readlane(__float_as_int(wt[0]), i & 63) : __builtin_amdgcn_readlane(__float_as_int(wt[1]), i & 63));
                if (i < parts) {
                    o.x = fmaf(ov[j].x, w, o.x);
                    o.y = fmaf(ov[j].y, w, o.y);
                }
            }
        }
        *reinterpret_cast<float2*>(sm + wave * S::kWaveBytes + 1024 + lane * 8) = o;
        lds_barrier();
        if (wave == 0) {
#pragma unroll
            for (int w = 1; w < WV; ++w) {
                const float2 x = *reinterpret_cast<const float2*>(sm + w * S::kWaveBytes + 1024 + lane * 8);
                o.x += x.x;
                o.y += x.y;
            }
            *reinterpret_cast<float2*>(out) = make_float2(o.x / lsum, o.y / lsum);
            if (lane == 0) __hip_atomic_store(p.counters + u, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

constexpr int kMaxDevices = 64;
// compute units of the current device (kept per device)
int compute_units() {
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    const bool keep = dev >= 0 && dev < kMaxDevices;
    if (keep) {
        const int c = cached[dev].load(std::memory_order_relaxed);
        if (c > 0) return c;
    }
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
    if (keep) cached[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

template <int BITS, int PT, int NB, int WV, int OCC, bool CS, bool FLUSH, bool UNEVEN, bool RAGGED>
hipError_t launch(DecodeParams p, hipStream_t stream) {
    using S = Shape<BITS, PT, NB, WV>;
    static_assert(S::kLds <= 160 * 1024 / OCC / 1280 * 1280, "workgroups per compute unit (LDS is given out in pieces of 1280 bytes)");
    static_assert(NB == 2 && PT <= 2, "two items in flight; masked tiles of a slot");
    if constexpr (RAGGED) {
        if (p.n_slices < 1) return hipErrorInvalidValue;
        p.one_round = p.n_slices <= (int64_t)compute_units() * OCC;
        decode_one_kernel<BITS, PT, NB, WV, OCC, CS, FLUSH, UNEVEN, RAGGED><<<(unsigned)p.n_slices, 64 * WV, 0, stream>>>(p);
        return hipGetLastError();
    }
    const int64_t units = (int64_t)p.batch * p.n_kv_heads;
    const int v_q = p.n_vq - (FLUSH ? kTileTokens : p.flushed_values);
    const int steps = OneHeadItems<BITS, FLUSH, UNEVEN>::steps((v_q + kTileTokens - 1) / kTileTokens, p.n_kq, v_q, p.n_kr);
    const int cus = compute_units();
    const int w = one_head_parts(units, steps, cus, std::min(p.part_stride, kOneHeadMaxParts), BITS == 2 ? 8 : 12);
    if (steps < 1 || units * w > 0x7fffffff) return hipErrorInvalidValue;
    p.unit_wgs = w;
    p.axis_len = steps / w;
    p.axis_rem = steps % w;
    p.one_round = units * w <= (int64_t)cus * OCC;
    decode_one_kernel<BITS, PT, NB, WV, OCC, CS, FLUSH, UNEVEN, RAGGED><<<(unsigned)(units * w), 64 * WV, 0, stream>>>(p);
    return hipGetLastError();
}

template <bool CS, bool FLUSH, bool UNEVEN, bool RAGGED = false>
hipError_t launch_bits(const DecodeParams& p, hipStream_t stream) {
    return p.bits == 2 ? launch<2, 2, 2, 4, 3, CS, FLUSH, UNEVEN, RAGGED>(p, stream) : launch<4, 1, 2, 4, 3, CS, FLUSH, UNEVEN, RAGGED>(p, stream);
}

}  // namespace

int one_head_compute_units() { return compute_units(); }

hipError_t launch_decode_one(const DecodeParams& p_in, hipStream_t stream) {
    DecodeParams p = p_in;
    p.flushed_values = 0;
    if (p.wave_desc) {
        if (p.n_q_heads != p.n_kv_heads || !p.unit_parts || p.flush_k || p.part_stride < 1) return hipErrorInvalidValue;
        return p.kg_shift > 0 ? launch_bits<true, false, false, true>(p, stream) : launch_bits<false, false, false, true>(p, stream);
    }
    if (p.n_q_heads != p.n_kv_heads || p.n_kq + p.n_kr != p.n_vq + p.n_vr || p.n_kq < p.n_vq || p.part_stride < 1) return hipErrorInvalidValue;
    const bool cs = p.kg_shift > 0;
    const QuantKeyParams* k = p.flush_k;
    const QuantValueParams* v = p.flush_v;
    if (k) {
        // the flushed tokens: one tile, the last quantised one, out of the rings right before the window
        if (!v || cs || p.n_kq != p.n_vq || k->n_tiles != 1 || v->n_tokens != kTileTokens || p.plan.tiles_a < 1 || p.n_kr < 1 ||
            k->first_tile != p.plan.tiles_a - 1 || v->first_token != (p.plan.tiles_a - 1) * kTileTokens)
            return hipErrorInvalidValue;
        return launch_bits<false, true, false>(p, stream);
    }
    if (v) {
        // ... or one value token, the last quantised one, out of the ring right before the others
        if (v->n_tokens != 1 || v->first_token != p.n_vq - 1 || p.n_vr >= p.cap_r) return hipErrorInvalidValue;
        p.flushed_values = 1;
    }
    if (v || p.n_kq != p.n_vq) return cs ? launch_bits<true, false, true>(p, stream) : launch_bits<false, false, true>(p, stream);
    return cs ? launch_bits<true, false, false>(p, stream) : launch_bits<false, false, false>(p, stream);
}

}  // namespace kivi
