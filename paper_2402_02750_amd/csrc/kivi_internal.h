// Internal declarations shared by the library's translation units (host side only).
// Nothing here is part of the ABI; see include/kivi.h for that.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "kivi.h"
#include "kivi_tiles_plan.h"

namespace kivi {

constexpr int kHeadDim = 128;
constexpr int kTileTokens = 32;        // tokens per code tile; a group of G = 32, 64 or 128 tokens covers 1, 2 or 4 tiles
constexpr int kMaxSplitTiles = 32;     // a context split covers at most 32 tiles (1024 tokens)
constexpr int kMfmaSplitTiles = 16;    // ... at most 16 tiles in the matrix-core family (4 per wavefront)
constexpr int kMaxRep = 8;             // query heads per kv-head handled by one launch
constexpr int kMaxRepTotal = 128;      // query heads per kv-head of a layout (wider groups take several launches)

// Source of fp16 rows for the quantise kernels: either a strided tensor or a ring buffer.
struct RowSource {
    const __half* base;   // element (b, h, t, c) at base[b*stride_b + h*stride_h + slot(t)*stride_t + c]
    int64_t stride_b, stride_h, stride_t;
    int32_t ring_start;   // slot(t) = (ring_start + t) % ring_cap when ring_cap > 0, else t
    int32_t ring_cap;
};

struct QuantKeyParams {
    RowSource src;
    uint32_t* codes;      // [b][h][cap_tiles][W]
    __half* scale;        // [b][h][cap_tiles][128]
    __half* zero;
    int32_t n_kv_heads, cap_tiles, bits;
    int32_t first_tile;   // destination tile index of source token 0
    int32_t n_tiles;
    int32_t batch;
    int32_t tiles_per_group;   // G / 32: 1, 2 or 4
};

struct QuantValueParams {
    RowSource src;
    uint32_t* codes;      // [b][h][cap_tiles][W]
    __half* scale;        // [b][h][cap_tokens][4]
    __half* zero;
    int32_t n_kv_heads, cap_tiles, bits;
    int32_t first_token;  // destination token index of source token 0 (any value)
    int32_t n_tokens;
    int32_t batch;
    int32_t group_blocks;      // G / 32: 32-channel blocks per group (1, 2 or 4)
};

// Copy fp16 rows of every (b, h) from strided tensors into residual rings: up to two (source,
// ring) pairs per launch (keys and values), the second is skipped when its n_tokens is 0.
struct CopyRowsParams {
    struct Job {
        const __half* src;    // element (b, h, t, c) at src[b*stride_b + h*stride_h + (src_t0 + t)*stride_t + c]
        int64_t stride_b, stride_h, stride_t;
        int32_t src_t0;
        __half* dst;          // [b][h][cap_r][128]
        int32_t dst_slot0;    // row t goes to slot (dst_slot0 + t) % cap_r
        int32_t n_tokens;
    } job[2];
    int32_t cap_r, n_kv_heads, batch;
};

// How the token axis [0, L) is cut into context splits (one workgroup each per (b, kv-head)).
// Region A = tiles [0, tiles_a): K and V both quantised.  Region B = tiles [tiles_a, tiles_total):
// at least one of K, V is fp16 there (5x the bytes per token), so its splits are shorter.
struct SplitPlan {
    int32_t tiles_a, tiles_total;
    int32_t tiles_per_split_a, tiles_per_split_b;
    int32_t n_splits_a, n_splits_b;
    __host__ __device__ int32_t n_splits() const { return n_splits_a + n_splits_b; }
};

struct DecodeParams {
    // cache
    const uint32_t* k_codes; const __half* k_scale; const __half* k_zero;
    const uint32_t* v_codes; const __half* v_scale; const __half* v_zero;
    const __half* k_resid; const __half* v_resid;
    // fused append (matrix-core family only; null otherwise): the rows of token length-1, [b][H_kv][128].
    // The kernel reads that token from here and writes it into the rings (which it may, then, modify).
    const __half* k_new; const __half* v_new;
    int32_t n_kq, n_vq, k_r_start, n_kr, v_r_start, n_vr;
    int32_t cap_tiles, cap_r;
    // problem
    const __half* q;        // [b][H_q][128]
    float* out;             // [b][H_q][128]
    int32_t* counters;      // workspace: [b][H_kv] finished-split counters (zero between calls)
    float* part_ml;         // workspace: [b][H_q][n_splits][2]  (max, sum)
    float* part_o;          // workspace: [b][H_q][n_splits][128]
    float softmax_scale;
    int32_t batch, n_q_heads, n_kv_heads, bits, length;
    // One launch serves query heads [q_head0, q_head0 + rep_here) of every kv-head's group, on the
    // kernel instantiation for rep_variant heads (>= rep_here; the surplus heads idle).  A group of
    // up to kMaxRep heads is one launch; a wider one (multi-query attention) takes several, all on
    // the kMaxRep instantiation so that they share one split plan.
    int32_t q_head0, rep_here, rep_variant;
    SplitPlan plan;
    // Persistent matrix-core kernel.  Work lies on a cost axis: unit u occupies [u * cost_unit,
    // (u + 1) * cost_unit): first its fp16-row chunks (cost_b each), then its all-quantised chunks
    // (cost 1 each).  Workgroup g of G owns the chunks that start in [g * T / G, (g + 1) * T / G),
    // T = units * cost_unit.
    int32_t total_chunks_a, total_chunks_b, cost_b, cost_unit;
    int64_t total_cost;
    // > 0: the matrix-core family runs as two launches (fp16 rows, then the all-quantised chunks); the
    // plan then has a single fp16-row split per unit (n_splits_b == 1).
    int32_t two_launches;
    // Batches whose sequences differ in length (null otherwise): per batch entry {n_q, n_r, k_r_start, v_r_start} in device memory (K
    // and V split alike).  The scalar counters and the plan above then describe the LONGEST sequence.
    const int32_t* seq_state;
    int32_t kg_shift;           // log2(G / 32): scales and zero-points are stored once per group (keys: row tile >> kg_shift;
                                // values: 4 >> kg_shift entries per token); > 0 runs on instantiations of its own
    int32_t head_groups;        // decode_tiles_kernel: runs of rep_here query heads per kv-head, each a unit of its own (the last may be shorter)
    // ... and the tables of such a batch: decode_tiles_kernel, wave_desc[4 g] = {first unit, first step in it, steps, 0} of workgroup g,
    // unit_parts[b] = steps before sequence b (kivi_tiles_plan.h); decode_one_kernel, an OneHeadSequence per sequence, and their
    // first workgroups.  n_slices: workgroups.
    const int32_t* wave_desc;
    const int32_t* unit_parts;
    int32_t n_slices;
    // Host side only (two-launch form): the residual flush of this decode step, to be carried out by
    // extra workgroups of the fp16-row launch instead of a launch of its own; null otherwise.
    const QuantKeyParams* flush_k;
    const QuantValueParams* flush_v;
    int32_t part_stride;        // workspace rows (parts) per (batch, query head)
    // decode_tiles_kernel: its first row_wgs workgroups hold the units' fp16 rows, row_split per unit; interval g of the axis of
    // all-quantised steps (of one unit, cut into unit_wgs intervals; unit_wgs = 0: of all units) has axis_len
    // steps, one more if g < axis_rem.
    int32_t row_wgs, row_split, unit_wgs, axis_len, axis_rem;
    int32_t flushed_values;     // decode_one_kernel: value tokens it quantises itself, the last of n_vq (0 or 1)
    int32_t one_round;          // decode_one_kernel: all its workgroups fit the device at once
    // a launch of the fp16 rows goes before decode_tiles_kernel (launch_ragged_rows): its part is the first of those that kernel
    // merges (maximum in the log2 domain, counted as finished)
    int32_t rows_for_tiles;
};

// launchers (each defined next to its kernels); they return hipGetLastError() after the launch
hipError_t launch_quantize_keys(const QuantKeyParams& p, hipStream_t stream);
hipError_t launch_quantize_values(const QuantValueParams& p, hipStream_t stream);
// key groups and value tokens of one residual flush in a single launch (either part may be empty)
hipError_t launch_flush_quantize(const QuantKeyParams& kp, const QuantValueParams& vp, hipStream_t stream);
hipError_t launch_copy_rows(const CopyRowsParams& p, hipStream_t stream);
// keys, values and residual rows of a prompt in one launch, where the bulk forms serve both (whole tiles, G = 32)
bool prefill_possible(const QuantKeyParams& kp, const QuantValueParams& vp);
hipError_t launch_prefill(const QuantKeyParams& kp, const QuantValueParams& vp, const CopyRowsParams& cp, hipStream_t stream);
hipError_t launch_decode_valu(const DecodeParams& p, hipStream_t stream);
hipError_t launch_decode_mfma(const DecodeParams& p, hipStream_t stream);
constexpr int kTilesMaxParts = 128;    // decode_tiles_kernel: parts of one (batch, kv-head, run of query heads) unit, at most
// decode_tiles_kernel (kivi_decode_tiles.hip); with two_launches > 0 the fp16-row launch goes before it
hipError_t launch_decode_tiles(DecodeParams p, hipStream_t stream);
// workgroups the device holds of it for a batch of different lengths
int tiles_resident_ragged(int bits, int rep, bool large_groups);
int tiles_max_parts(int bits, int rep);       // parts of one unit that it merges, at most
// decode_one_kernel (kivi_decode_one.hip): one query head per kv-head, n_kq >= n_vq, one launch
// (with p.wave_desc: a batch of different lengths, G as one likes; wave_desc and unit_parts are the two tables of RaggedTables,
// n_slices all workgroups)
hipError_t launch_decode_one(const DecodeParams& p, hipStream_t stream);
int one_head_compute_units();
hipError_t launch_residual_rows(const DecodeParams& p, hipStream_t stream);
// Batches of different lengths before decode_tiles_kernel: fp16 rows, append, flush and tables (kivi_ragged_rows.hip).
// What the kernel writes for the second launch, in device memory: every sequence's counters (as seq_state), the steps before it, and the
// intervals of the axis of steps.
struct RaggedTables {
    int32_t *seq_state, *before, *intervals;
    int32_t n_intervals, axis_len, axis_rem, units_per_sequence;
    // decode_one_kernel instead: an OneHeadSequence per sequence, longest first, and the first workgroups once more on their own
    int32_t *one_head, *first_wg;
};
constexpr int kInlineSequences = 192;  // sequences whose counters fit the kernel's arguments (4096 bytes)
constexpr int kDeviceTableSequences = 4096;    // ... of which the launch makes the tables, at most (8 bytes of LDS each)
// p.rows_for_tiles: a batch of one length, no tables; seq and flush null, n_flush the batch, if it flushes a tile, or 0.  Otherwise
// seq: the counters in host memory, at most kInlineSequences of them, `flush` the n_flush sequences whose last quantised tile (G = 32) is still in
// the rings; null: the counters are in p.seq_state already, nothing is flushed, and tables may be null (there already).  max_tiles: of fp16 rows, of
// any sequence.
// one_head (tables->one_head): no fp16 rows; `sequences` in the order of the table, seq and flush in that order too.
hipError_t launch_ragged_one_head(const DecodeParams& p, const OneHeadSequence* sequences, const uint8_t* flush, int n_flush, const RaggedTables& tables,
                                  hipStream_t stream);
hipError_t launch_ragged_rows(const DecodeParams& p, int max_tiles, const int32_t* seq, const uint8_t* flush, int n_flush, const RaggedTables* tables,
                              hipStream_t stream);
// the same launch with extra workgroups that quantise the key group(s) and value tokens of a residual
// flush (G = 32 only: hipErrorNotSupported otherwise, nothing launched)
hipError_t launch_rows_and_flush(const DecodeParams& p, const QuantKeyParams& kp, const QuantValueParams& vp, hipStream_t stream);
hipError_t launch_merge(const DecodeParams& p, hipStream_t stream);
hipError_t launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t stream);

// Chunk length (tiles) of all-quantised chunks and resident workgroups of the matrix-core instantiation
// that serves (bits, query heads per kv-head); the split planner and the kernel must agree on both.
struct MfmaGeometry { int chunk_tiles, resident_workgroups; };
MfmaGeometry mfma_geometry(int bits, int rep);

}  // namespace kivi
