// Two and more query heads per kv-head, and batches of sequences of different lengths: the first of a step's two launches (KIVI Equation 4, the X_R terms, and Algorithm 1
// Decoding).  Its workgroups have one of three roles:
//   flush   (G = 32) one per unit of a sequence whose oldest 32 tokens leave the window: one wavefront quantises the keys, one the values
//   tables  one: the second launch's intervals into the workspace, and the sequences' counters, where they are arguments
//   rows    one per (batch, kv-head) and run of up to 16 query heads: attention over the fp16 rows, and the append of the new token
// The roles do not wait for each other: the rows leave out what is flushed, and the flush reads slots that the append does not
// write (a ring never is full before an append).
//
// What this replaces: a launch per run of equal sequences that flush (4.9 us each), a copy of the tables from host memory (a launch of
// its own on the device, 4.6 us) and a launch for the rows (15.2 us; 512 units of four heads, 128 to 159 rows each).
//
// Rows: one wavefront per tile of 32 tokens, both key and value rows requested up front.  Keys are matrix operands as they are, the
// instruction's columns are query heads (no remainders: both factors are fp16).  Lane kb gets the logits of tokens 8 kb .. 8 kb + 7,
// whose value rows it holds, channels 8 n ..: 32 byte permutes turn those 8 x 8 numbers into the operands whose rows are channels
// 8 n + e.  Probabilities enter as three fp16 numbers that add up to all 24 bits.  (With dot products on the vector unit, as
// residual_rows_kernel has them for one and two heads, each head costs 300 vector instructions more.)
// Bound: latency -- launch, counters, rows, matrix unit, merge of the tiles in LDS, a chain that all wavefronts run at once.
// Whole steps, before / with this launch: 64 sequences of 500-8000 tokens, 32 / 8 heads 81.6 / 69.5 us; 8 of them 37.1 / 24.6; 4 of 100-300
// tokens 19.7 / 12.1; 64 / 8 heads, 4 of 4000-16 000 53.0 / 35.2, 28 / 4, 4 bits, 32 of 400-5000 68.5 / 49.2; 200 sequences, counters copied, 155 / 112.
// Batches of one length, three and more heads, the two-launch form (kOneLength; before: the rows by decode_tiles_kernel, 53 KB of LDS a workgroup, or by
// rows_flush_kernel, and with five and more heads a launch for the flush): 64 x 32 / 8 heads, 2000 tokens 43.9 -> 39.7 us, with a flush 45.2 ->
// 40.3, 4096 tokens 64.6 -> 58.8; 32 x 64 / 8, 2047 39.6 -> 33.5; 16 x 64 / 8, 4095, 4 bits 50.2 -> 43.0; 32 x 28 / 4, 3000, 4 bits 34.9 -> 29.3.
// Forms that went run by run before: G = 64, 64 x 32 / 8 heads 787 / 71 us; 71 / 1 heads, 16 sequences 399 / 41.
#include "kivi_internal.h"
#include "kivi_quantize_tile.h"
#include "kivi_tiles_plan.h"

#include <hip/hip_fp16.h>

#include <algorithm>

namespace kivi {
namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

union Frag {
    half8 h;
    half2v p[4];
    uint32_t r[4];
    uint4v v;
};

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kProbExp = 12.f;               // probabilities enter as p 2^12: the smallest parts stay above fp16's subnormals
constexpr int kPartFloats = kHeadDim + 4;      // o[128], m, l

struct RaggedRowsParams : DecodeParams {
    FastDiv by_kv_heads, by_chunks;
    int32_t n_chunks, chunk_heads;             // runs of query heads of a kv-head that the rows take at once
    int32_t n_flush;                           // flush workgroups
    RaggedTables tables;
    int4 seq[kInlineSequences];                // n_q, n_r, k_r_start, v_r_start after the step
    uint8_t flush[kInlineSequences];           // which of them flush
    uint8_t sequence[kInlineSequences];        // one head: the batch entries that `seq` is of (n_r | parts << 16 there)
};
static_assert(sizeof(RaggedRowsParams) <= 4096, "kernel arguments");

__device__ __forceinline__ int ring_slot(int start, int i, int cap) {
    int s = start + i;
    s -= (s >= cap) ? cap : 0;
    return s;
}
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
__device__ __forceinline__ half2v pack_rtz(float a, float b) { return __builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(a, b)); }

// Where a sequence's counters are: among the arguments, in p.seq_state (then nothing is flushed here), or p's own for all of them
// (a batch of one length; then there are no tables)
constexpr int kInArguments = 0, kInMemory = 1, kOneLength = 2;

template <int BITS, int SOURCE>
__global__ __launch_bounds__(1024) void ragged_rows_kernel(RaggedRowsParams p) {
    extern __shared__ __align__(16) float sm_dyn[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_waves = blockDim.x >> 6;
    const int n = lane & 15, kb = lane >> 4;
    int at = blockIdx.x;
    const int4 all = make_int4(p.n_kq, p.n_kr, p.k_r_start, p.v_r_start);       // kOneLength
    if constexpr (SOURCE != kInMemory) {
        if (at < p.n_flush) {
            const int f = p.by_kv_heads.of(at), i = SOURCE == kOneLength ? f : p.flush[f], b = SOURCE != kOneLength && p.tables.one_head ? p.sequence[i] : i;
            const int64_t unit = (int64_t)b * p.n_kv_heads + (at - f * p.n_kv_heads);
            const int4 st = SOURCE == kOneLength ? all : p.seq[i];
            const int64_t tile = unit * p.cap_tiles + st.x / kTileTokens - 1;
            if (wave == 0) tile::flush_keys<BITS>(p, unit, tile, st.z, lane);
            if (wave == min(1, n_waves - 1)) tile::flush_values<BITS>(p, unit, tile, st.w, lane);
            return;
        }
        at -= p.n_flush;
    }
    const bool makes_tables = SOURCE == kInArguments || (SOURCE == kInMemory && p.tables.intervals);
    if (makes_tables) {
        if (at == 0) {
            const RaggedTables& t = p.tables;
            int* before = reinterpret_cast<int*>(sm_dyn);               // [batch]
            int* steps = before + p.batch;
            const bool one_head = SOURCE == kInArguments && t.one_head != nullptr;
            if (wave == 0) {
                int sum = 0;
                for (int b0 = 0; b0 < p.batch; b0 += 64) {
                    const int b = b0 + lane;
                    int mine = 0;
                    if (b < p.batch) {
                        int4 st;
                        if constexpr (SOURCE == kInArguments) st = p.seq[b];
                        else st = reinterpret_cast<const int4*>(p.seq_state)[b];
                        if (one_head) {
                            mine = (st.y >> 16) * p.n_kv_heads;         // (of the workgroups' axis)
                        } else {
                            if (SOURCE == kInArguments) reinterpret_cast<int4*>(t.seq_state)[b] = st;
                            steps[b] = ragged_steps(st.x);
                            mine = steps[b] * t.units_per_sequence;
                        }
                    }
                    int upto = mine;                                     // of this and the lanes before
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int x = __shfl_up(upto, d);
                        if (lane >= d) upto += x;
                    }
                    if (b < p.batch) {
                        before[b] = sum + upto - mine;
                        if (one_head) {
                            const int4 st = p.seq[b];
                            const int n_r = st.y & 0xffff;
                            t.first_wg[b] = before[b];
                            reinterpret_cast<OneHeadSequence*>(t.one_head)[b] = OneHeadSequence{before[b], p.sequence[b], st.y >> 16, st.x, n_r, st.z, st.w,
                                                                                                OneHeadItems<BITS, false, false>::steps(st.x / kTileTokens, st.x, st.x, n_r)};
                        } else {
                            t.before[b] = before[b];
                        }
                    }
                    sum += __shfl(upto, 63);
                }
            }
            if (one_head) return;
            __syncthreads();
            const StepAxis axis{t.axis_len, t.axis_rem};
            for (int g = tid; g < t.n_intervals; g += blockDim.x)
                reinterpret_cast<int4*>(t.intervals)[g] = __builtin_bit_cast(int4, ragged_interval(before, steps, p.batch, t.units_per_sequence, axis, g));
            return;
        }
        at -= 1;
    }
    // ---- rows ----
    const int unit_i = p.by_chunks.of(at), chunk = at - unit_i * p.n_chunks;
    const int b = p.by_kv_heads.of(unit_i), kvh = unit_i - b * p.n_kv_heads;
    const int64_t unit = unit_i;
    const int rep_total = p.n_q_heads / p.n_kv_heads, h0 = p.q_head0 + chunk * p.chunk_heads;
    const int heads = min(p.chunk_heads, min(rep_total, p.q_head0 + p.rep_here) - h0);
    int4 st;
    if constexpr (SOURCE == kInArguments) st = p.seq[b];
    else if constexpr (SOURCE == kOneLength) st = all;
    else st = reinterpret_cast<const int4*>(p.seq_state)[b];
    const int n_q = st.x, last = st.x + st.y - 1, tt = n_q + wave * kTileTokens;
    const int64_t q_row0 = (int64_t)b * p.n_q_heads + (int64_t)kvh * rep_total + h0;
    float* part = sm_dyn + (int64_t)wave * p.chunk_heads * kPartFloats;
    if (tt <= last) {
        const __half* k_new = p.k_new ? p.k_new + unit * kHeadDim : nullptr;
        const __half* v_new = p.v_new ? p.v_new + unit * kHeadDim : nullptr;
        const __half* k_ring = p.k_resid + unit * p.cap_r * kHeadDim;
        const __half* v_ring = p.v_resid + unit * p.cap_r * kHeadDim;
        Frag kr[2][4], vr[8], q[4];
        // row m of the half-th instruction: token 8 (m / 4) + 4 half + m % 4 (rows past the end re-read the last one)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int t = min(tt + (n >> 2) * 8 + 4 * half + (n & 3), last);
            const __half* src = k_new && t == last ? k_new : k_ring + (int64_t)ring_slot(st.z, t - n_q, p.cap_r) * kHeadDim;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) kr[half][cb].v = *reinterpret_cast<const uint4v*>(src + cb * 32 + kb * 8);
        }
        const __half* q_row = p.q + (q_row0 + min(n, heads - 1)) * kHeadDim + kb * 8;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) q[cb].v = *reinterpret_cast<const uint4v*>(q_row + cb * 32);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t = min(tt + kb * 8 + i, last);
            const __half* src = v_new && t == last ? v_new : v_ring + (int64_t)ring_slot(st.w, t - n_q, p.cap_r) * kHeadDim;
            vr[i].v = *reinterpret_cast<const uint4v*>(src + n * 8);
        }
        // the wavefront of the newest token's tile puts its rows into the rings
        if (k_new && chunk == 0 && p.q_head0 == 0 && last < tt + kTileTokens && lane < 32) {
            const bool is_v = lane >= 16;
            const int slot = ring_slot(is_v ? st.w : st.z, last - n_q, p.cap_r);
            const uint4v row = *reinterpret_cast<const uint4v*>((is_v ? v_new : k_new) + n * 8);
            *reinterpret_cast<uint4v*>(const_cast<__half*>(is_v ? v_ring : k_ring) + (int64_t)slot * kHeadDim + n * 8) = row;
        }
        float x[8], mx = -INFINITY;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float4v d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) d = __builtin_amdgcn_mfma_f32_16x16x32_f16(kr[half][cb].h, q[cb].h, d, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[4 * half + i] = tt + 8 * kb + 4 * half + i <= last ? d[i] * (p.softmax_scale * kLog2e) : -INFINITY;
                mx = fmaxf(mx, x[4 * half + i]);
            }
        }
        mx = max_rows(mx);                             // -inf only where every token's logit is: such a tile counts for nothing
        const float ref = mx == -INFINITY ? 0.f : mx;
        float l = 0.f;
        Frag hi, mid, lo;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float pr[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                pr[k] = __builtin_amdgcn_exp2f(x[2 * r + k] - ref + kProbExp);
                l += pr[k];
            }
            hi.p[r] = pack_rtz(pr[0], pr[1]);          // 11 + 11 + 2 bits; the remainders are exact
            pr[0] -= (float)hi.p[r][0]; pr[1] -= (float)hi.p[r][1];
            mid.p[r] = pack_rtz(pr[0], pr[1]);
            pr[0] -= (float)mid.p[r][0]; pr[1] -= (float)mid.p[r][1];
            lo.p[r] = pack_rtz(pr[0], pr[1]);
        }
        l = add_rows(l);
        float4v o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // rows: channels 8 n + e; contraction: this lane's eight tokens
            Frag a;
#pragma unroll
            for (int r = 0; r < 4; ++r) a.r[r] = __builtin_amdgcn_perm(vr[2 * r + 1].r[e / 2], vr[2 * r].r[e / 2], e & 1 ? 0x07060302u : 0x05040100u);
            o[e] = float4v{0.f, 0.f, 0.f, 0.f};
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, lo.h, o[e], 0, 0, 0);
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, mid.h, o[e], 0, 0, 0);
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, hi.h, o[e], 0, 0, 0);
        }
        if (n < heads) {
            float* dst = part + n * kPartFloats;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *reinterpret_cast<float4v*>(dst + (4 * kb + i) * 8) = float4v{o[0][i], o[1][i], o[2][i], o[3][i]};
                *reinterpret_cast<float4v*>(dst + (4 * kb + i) * 8 + 4) = float4v{o[4][i], o[5][i], o[6][i], o[7][i]};
            }
            if (kb == 0) {
                dst[kHeadDim] = mx - kProbExp;
                dst[kHeadDim + 1] = l;
            }
        }
    }
    __syncthreads();
    // the tiles of the unit: part 0 of every query head (maximum in the log2 domain)
    const int n_tiles = min((last - n_q) / kTileTokens + 1, n_waves);
    for (int idx = tid; idx < heads * (kHeadDim / 4); idx += blockDim.x) {
        const int hh = idx / (kHeadDim / 4), c = idx % (kHeadDim / 4) * 4;
        const float* src = sm_dyn + hh * kPartFloats;
        const int stride = p.chunk_heads * kPartFloats;
        float m = -INFINITY, l = 0.f;
        for (int w = 0; w < n_tiles; ++w) m = fmaxf(m, src[w * stride + kHeadDim]);
        float4v o = {0.f, 0.f, 0.f, 0.f};
        const float ref = m == -INFINITY ? 0.f : m;
        for (int w = 0; w < n_tiles; ++w) {
            const float f = __builtin_amdgcn_exp2f(src[w * stride + kHeadDim] - ref);
            l = fmaf(src[w * stride + kHeadDim + 1], f, l);
            const float4v x = *reinterpret_cast<const float4v*>(src + w * stride + c);
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = fmaf(x[k], f, o[k]);
        }
        const int64_t row = (q_row0 + hh) * p.part_stride;
        *reinterpret_cast<float4v*>(p.part_o + row * kHeadDim + c) = o;
        if (c == 0) *reinterpret_cast<float2*>(p.part_ml + row * 2) = make_float2(m, l);
    }
    if (SOURCE == kOneLength && tid == 0) __hip_atomic_fetch_add(p.counters + unit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (one of the parts that decode_tiles_kernel counts)
}

}  // namespace

hipError_t launch_ragged_one_head(const DecodeParams& params, const OneHeadSequence* sequences, const uint8_t* flush, int n_flush, const RaggedTables& tables,
                                  hipStream_t stream) {
    if (params.batch > kInlineSequences || !tables.one_head || !tables.first_wg) return hipErrorInvalidValue;
    RaggedRowsParams p{};
    static_cast<DecodeParams&>(p) = params;
    p.by_kv_heads = FastDiv::by(p.n_kv_heads);
    p.n_flush = n_flush * p.n_kv_heads;
    p.tables = tables;
    for (int i = 0; i < p.batch; ++i) {
        const OneHeadSequence& s = sequences[i];
        if (s.n_r > 0xffff || s.parts > 0x7fff) return hipErrorInvalidValue;
        p.seq[i] = make_int4(s.n_q, s.n_r | s.parts << 16, s.k_start, s.v_start);
        p.sequence[i] = (uint8_t)s.sequence;
    }
    std::copy(flush, flush + n_flush, p.flush);
    const unsigned grid = (unsigned)(p.n_flush + 1), lds = sizeof(int) * 2 * p.batch;
    if (p.bits == 2) ragged_rows_kernel<2, kInArguments><<<grid, 128, lds, stream>>>(p);
    else ragged_rows_kernel<4, kInArguments><<<grid, 128, lds, stream>>>(p);
    return hipGetLastError();
}

hipError_t launch_ragged_rows(const DecodeParams& params, int max_tiles, const int32_t* seq, const uint8_t* flush, int n_flush, const RaggedTables* tables,
                              hipStream_t stream) {
    const int rep_total = params.n_q_heads / params.n_kv_heads, heads = std::min(params.rep_here, rep_total - params.q_head0);
    const int64_t units = (int64_t)params.batch * params.n_kv_heads;
    const bool one_length = params.rows_for_tiles > 0, in_arguments = !one_length && seq != nullptr;
    // (max_tiles and heads: as residual_rows_possible has them)
    if ((tables && tables->one_head) || max_tiles < 1 || max_tiles > 16 || heads < 1 || params.part_stride < 1) return hipErrorInvalidValue;
    if (one_length ? seq || tables || heads > 8 || (n_flush != 0 && n_flush != params.batch) || params.n_kq != params.n_vq || params.n_kr < 1
                   : in_arguments ? params.batch > kInlineSequences || !tables
                                  : !params.seq_state || n_flush > 0 || (tables && params.batch > kDeviceTableSequences))
        return hipErrorInvalidValue;
    RaggedRowsParams p{};
    static_cast<DecodeParams&>(p) = params;
    p.chunk_heads = rows_chunk_heads(heads, max_tiles);
    p.n_chunks = (heads + p.chunk_heads - 1) / p.chunk_heads;
    if (p.chunk_heads * max_tiles > kRowsChunkTiles) return hipErrorInvalidValue;
    if (one_length && p.n_chunks != 1) return hipErrorInvalidValue;      // (a unit's rows are counted as one part)
    p.rep_here = heads;
    p.by_kv_heads = FastDiv::by(p.n_kv_heads);
    p.by_chunks = FastDiv::by(p.n_chunks);
    p.n_flush = n_flush * p.n_kv_heads;
    const int64_t grid = units * p.n_chunks + (tables ? 1 : 0) + p.n_flush;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    size_t lds = (size_t)max_tiles * p.chunk_heads * kPartFloats * sizeof(float);
    const unsigned threads = 64 * max_tiles;
    if (tables) {
        p.tables = *tables;
        lds = std::max(lds, sizeof(int) * 2 * p.batch);
    }
    if (in_arguments) {
        for (int b = 0; b < p.batch; ++b) p.seq[b] = make_int4(seq[4 * b], seq[4 * b + 1], seq[4 * b + 2], seq[4 * b + 3]);
        std::copy(flush, flush + n_flush, p.flush);
        if (p.bits == 2) ragged_rows_kernel<2, kInArguments><<<(unsigned)grid, threads, lds, stream>>>(p);
        else ragged_rows_kernel<4, kInArguments><<<(unsigned)grid, threads, lds, stream>>>(p);
    } else if (one_length) {
        if (p.bits == 2) ragged_rows_kernel<2, kOneLength><<<(unsigned)grid, threads, lds, stream>>>(p);
        else ragged_rows_kernel<4, kOneLength><<<(unsigned)grid, threads, lds, stream>>>(p);
    } else {
        ragged_rows_kernel<2, kInMemory><<<(unsigned)grid, threads, lds, stream>>>(p);      // (the bits are the flush's)
    }
    return hipGetLastError();
}

}  // namespace kivi
