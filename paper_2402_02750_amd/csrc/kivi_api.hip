// Host side of the C ABI (include/kivi.h): argument validation, split planning, launches.
// No allocation, no synchronisation; the only state kept between calls is, per device, the address
// of the static scratch array below (and the occupancy answers next to the decode kernels).
#include "kivi_internal.h"
#include "kivi_tiles_plan.h"

#include <algorithm>
#include <vector>
#include <atomic>

namespace kivi {
namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_layout(const kivi_layout_t* l) {
    if (!l) return KIVI_ERR_INVALID_ARG;
    if (l->batch < 1 || l->n_q_heads < 1 || l->n_kv_heads < 1) return KIVI_ERR_INVALID_ARG;
    if (l->batch > 65535 || l->n_kv_heads > 65535) return KIVI_ERR_INVALID_ARG;
    if (l->n_q_heads % l->n_kv_heads != 0) return KIVI_ERR_INVALID_ARG;
    if (l->residual < 0 || l->cap_q_tokens < 0 || l->cap_r_tokens < 0) return KIVI_ERR_INVALID_ARG;
    if (l->decode_path < KIVI_DECODE_AUTO || l->decode_path > KIVI_DECODE_MFMA_TWO) return KIVI_ERR_INVALID_ARG;
    if (l->head_dim != kHeadDim) return KIVI_ERR_UNSUPPORTED;
    if (l->bits != 2 && l->bits != 4) return KIVI_ERR_UNSUPPORTED;
    if (l->group != 32 && l->group != 64 && l->group != 128) return KIVI_ERR_UNSUPPORTED;
    if (l->residual % l->group != 0) return KIVI_ERR_INVALID_ARG;          // Section 3.3: G | R
    if (l->cap_q_tokens % l->group != 0 || l->cap_r_tokens % kTileTokens != 0) return KIVI_ERR_INVALID_ARG;
    if (l->cap_r_tokens < l->residual + l->group) return KIVI_ERR_INVALID_ARG;
    const int rep = l->n_q_heads / l->n_kv_heads;
    if (rep > kMaxRepTotal) return KIVI_ERR_UNSUPPORTED;
    return KIVI_OK;
}

int check_cache(const kivi_layout_t* l, const kivi_cache_t* c) {
    if (!c) return KIVI_ERR_INVALID_ARG;
    const void* ptrs[8] = {c->k_codes, c->k_scale, c->k_zero, c->v_codes,
                           c->v_scale, c->v_zero, c->k_resid, c->v_resid};
    for (const void* p : ptrs)
        if (!p || !aligned16(p)) return KIVI_ERR_INVALID_ARG;
    if (c->n_kq < 0 || c->n_vq < 0 || c->n_kr < 0 || c->n_vr < 0) return KIVI_ERR_INVALID_ARG;
    if (c->n_kq % l->group != 0) return KIVI_ERR_INVALID_ARG;
    if (c->n_kq > l->cap_q_tokens || c->n_vq > l->cap_q_tokens) return KIVI_ERR_INVALID_ARG;
    if (c->n_kr > l->cap_r_tokens || c->n_vr > l->cap_r_tokens) return KIVI_ERR_INVALID_ARG;
    if (c->k_r_start < 0 || c->k_r_start >= l->cap_r_tokens) return KIVI_ERR_INVALID_ARG;
    if (c->v_r_start < 0 || c->v_r_start >= l->cap_r_tokens) return KIVI_ERR_INVALID_ARG;
    return KIVI_OK;
}

int check_source(const void* x, int64_t sb, int64_t sh, int64_t st) {
    if (!x || !aligned16(x)) return KIVI_ERR_INVALID_ARG;
    if (sb < 0 || sh < 0 || st < kHeadDim) return KIVI_ERR_INVALID_ARG;
    if ((sb | sh | st) & 7) return KIVI_ERR_INVALID_ARG;          // keeps every row 16-byte aligned
    return KIVI_OK;
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The workspace starts with four finished-split counters per (batch, kv-head) -- one per quarter of
// the kv-head's query heads, should a launch serve parts of the group as units of their own -- padded
// to 256 bytes.
size_t counter_bytes(const kivi_layout_t* l) {
    // one counter per unit of the work axis: up to 4 parts of a kv-head's query heads (head split), or
    // one per run of 4 heads of a group wider than kMaxRep
    const int groups = std::max(4, ceil_div(l->n_q_heads / std::max(l->n_kv_heads, 1), 4));
    return ((size_t)l->batch * l->n_kv_heads * groups * sizeof(int32_t) + 255) / 256 * 256;
}

// Room for the per-sequence counters of a batch of different lengths (16 bytes per sequence, padded
// to 256 bytes); the ragged entry points keep them behind the split counters.
size_t seq_state_bytes(const kivi_layout_t* l) {
    return ((size_t)l->batch * 4 * sizeof(int32_t) + 255) / 256 * 256;
}

// Room for the tables of the second launch of such a batch, behind the counters: 16 bytes per workgroup (at most kMaxSlices) and 8
// bytes per (batch, kv-head) unit, of which 4 bytes per sequence are used.
constexpr int kMaxSlices = 4096;
constexpr int64_t kMaxSliceUnits = 65536;
size_t slice_table_bytes(const kivi_layout_t* l) {
    const int64_t units = std::min<int64_t>((int64_t)l->batch * l->n_kv_heads, kMaxSliceUnits);
    size_t bytes = (size_t)kMaxSlices * 16 + (size_t)units * 8;
    // decode_one_kernel's tables lie there and in the counters' place: 36 bytes per sequence, more with one kv-head and 5400 sequences
    if (l->n_q_heads == l->n_kv_heads) bytes = std::max(bytes, (size_t)l->batch * 36 - std::min((size_t)l->batch * 36, seq_state_bytes(l)));
    return (bytes + 255) / 256 * 256;
}

// Upper bound of the number of context splits for any cache state of this layout.
// Both planners below give every all-quantised split at least 4 tiles (the matrix-core family 8 or
// 16), and every split with fp16 rows at least one tile; enqueue_attention checks the actual count
// against the workspace before it launches.
int max_splits(const kivi_layout_t* l) {
    const int tiles_q = l->cap_q_tokens / kTileTokens, tiles_r = l->cap_r_tokens / kTileTokens;
    return (tiles_q + 3) / 4 + tiles_r + 2;
}

// `mfma`: plan for the persistent matrix-core kernel (fixed chunk length, resident workgroups known);
// otherwise for the vector-ALU family.
// `two_launches` (matrix-core family only): a single fp16-row split per unit, served by a launch of its own.
SplitPlan plan_splits(const kivi_layout_t* l, const kivi_cache_t* c, bool mfma, bool two_launches = false) {
    SplitPlan s{};
    const int length = c->n_kq + c->n_kr;
    s.tiles_a = std::min(c->n_kq, c->n_vq) / kTileTokens;
    s.tiles_total = ceil_div(length, kTileTokens);
    const int64_t units = (int64_t)l->batch * l->n_kv_heads;
    const int rep = std::min(l->n_q_heads / l->n_kv_heads, kMaxRep);      // heads per launch (wider groups: several launches)
    const int tiles_b = s.tiles_total - s.tiles_a;
    int tps_b_max;
    if (mfma) {
        // The kernel always walks full chunks (shorter ones would only re-read masked tiles).  The
        // natural fp16-row chunk is 4 tiles, one per wavefront; shorter ones when there would be
        // fewer chunks than resident workgroups.
        const MfmaGeometry g = mfma_geometry(l->bits, rep);
        s.tiles_per_split_a = g.chunk_tiles;
        tps_b_max = (int)std::max<int64_t>(1, std::min<int64_t>(4, units * tiles_b / g.resident_workgroups));
        if (two_launches) tps_b_max = std::max(tiles_b, 1);
    } else {
        // Aim at ~16 workgroups per compute unit in flight over the whole grid so the 256 CUs stay
        // busy through the tail, but keep splits long enough that the per-split partial results
        // (520 B per query head) stay a small fraction of the bytes a split streams.
        const int64_t target_wgs = 4096;
        int tps = (int)std::min<int64_t>(kMaxSplitTiles, ((int64_t)s.tiles_a * units + target_wgs - 1) / target_wgs);
        tps = std::max(tps, std::min(kMaxSplitTiles, 4 * rep));
        s.tiles_per_split_a = std::max(1, std::min(tps, kMaxSplitTiles));
        // fp16 rows cost 512 B per token against 96 B (2-bit) or 160 B (4-bit)
        const int packed_per_tile = kTileTokens * 2 * (kHeadDim * l->bits / 8 + 16);
        const int fp16_per_tile = kTileTokens * 2 * kHeadDim * 2;
        tps_b_max = std::max(1, std::min(8, s.tiles_per_split_a * packed_per_tile / fp16_per_tile));
    }
    s.n_splits_b = ceil_div(tiles_b, tps_b_max);
    s.tiles_per_split_b = s.n_splits_b ? ceil_div(tiles_b, s.n_splits_b) : 1;     // even out the pieces
    s.n_splits_a = ceil_div(s.tiles_a, s.tiles_per_split_a);
    return s;
}

int hip_status(hipError_t e) { return e == hipSuccess ? KIVI_OK : KIVI_ERR_HIP; }

QuantKeyParams key_quant_params(const kivi_layout_t* l, const kivi_cache_t* c, const RowSource& src, int n_tokens) {
    QuantKeyParams p{};
    p.src = src;
    p.codes = static_cast<uint32_t*>(c->k_codes);
    p.scale = static_cast<__half*>(c->k_scale);
    p.zero = static_cast<__half*>(c->k_zero);
    p.n_kv_heads = l->n_kv_heads; p.cap_tiles = l->cap_q_tokens / kTileTokens; p.bits = l->bits;
    p.first_tile = c->n_kq / kTileTokens; p.n_tiles = n_tokens / kTileTokens; p.batch = l->batch;
    p.tiles_per_group = l->group / kTileTokens;
    return p;
}

QuantValueParams value_quant_params(const kivi_layout_t* l, const kivi_cache_t* c, const RowSource& src, int n_tokens) {
    QuantValueParams p{};
    p.src = src;
    p.codes = static_cast<uint32_t*>(c->v_codes);
    p.scale = static_cast<__half*>(c->v_scale);
    p.zero = static_cast<__half*>(c->v_zero);
    p.n_kv_heads = l->n_kv_heads; p.cap_tiles = l->cap_q_tokens / kTileTokens; p.bits = l->bits;
    p.first_token = c->n_vq; p.n_tokens = n_tokens; p.batch = l->batch;
    p.group_blocks = l->group / kTileTokens;
    return p;
}

int enqueue_key_quant(const kivi_layout_t* l, const kivi_cache_t* c, const RowSource& src, int n_tokens,
                      hipStream_t hs) {
    return hip_status(launch_quantize_keys(key_quant_params(l, c, src, n_tokens), hs));
}

int enqueue_value_quant(const kivi_layout_t* l, const kivi_cache_t* c, const RowSource& src, int n_tokens,
                        hipStream_t hs) {
    return hip_status(launch_quantize_values(value_quant_params(l, c, src, n_tokens), hs));
}

}  // namespace
}  // namespace kivi

using namespace kivi;

namespace {

// How many of the oldest residual tokens each policy moves into the quantised part (host logic).
int plan_flush(const kivi_layout_t* l, const kivi_cache_t* c, int32_t policy, int* n_key, int* n_value) {
    const int G = l->group, R = l->residual;
    int nk = 0, nv = 0;
    if (policy == KIVI_FLUSH_WINDOW) {
        if (c->n_kr != c->n_vr || c->n_kq != c->n_vq) return KIVI_ERR_INVALID_ARG;   // symmetric policy
        while (c->n_kr - nk >= R + G) nk += G;
        nv = nk;
    } else {
        if (R > 0 && c->n_kr == R) nk = R;                 // Algorithm 1: len(X_Kr) == R
        if (c->n_vr > R) nv = c->n_vr - R;                 // Algorithm 1: len(X_Vr) > R
    }
    if ((int64_t)c->n_kq + nk > l->cap_q_tokens || (int64_t)c->n_vq + nv > l->cap_q_tokens)
        return KIVI_ERR_INVALID_ARG;
    *n_key = nk;
    *n_value = nv;
    return KIVI_OK;
}

// Quantise the oldest nk residual keys and nv residual values out of the rings (one launch; either
// count may be 0) and advance the cache counters (`launch` false: the counters only).
int enqueue_flush(const kivi_layout_t* l, kivi_cache_t* c, int nk, int nv, hipStream_t hs, bool launch = true) {
    const int64_t sh = (int64_t)l->cap_r_tokens * kHeadDim, sb = sh * l->n_kv_heads;
    if (launch && (nk > 0 || nv > 0)) {
        const RowSource ksrc{static_cast<const __half*>(c->k_resid), sb, sh, kHeadDim, c->k_r_start, l->cap_r_tokens};
        const RowSource vsrc{static_cast<const __half*>(c->v_resid), sb, sh, kHeadDim, c->v_r_start, l->cap_r_tokens};
        if (int s = hip_status(launch_flush_quantize(key_quant_params(l, c, ksrc, nk), value_quant_params(l, c, vsrc, nv), hs)))
            return s;
    }
    c->n_kq += nk; c->n_kr -= nk; c->k_r_start = (c->k_r_start + nk) % l->cap_r_tokens;
    c->n_vq += nv; c->n_vr -= nv; c->v_r_start = (c->v_r_start + nv) % l->cap_r_tokens;
    return KIVI_OK;
}

// Host checks shared by the attention entry points (the cache counts are those the kernel will see).
// any_state: the workspace must hold the parts of any cache state of the layout (the documented
// size); otherwise only a pointer check -- enqueue_attention checks the state's own need.
int check_attention_args(const kivi_layout_t* l, const kivi_cache_t* c, const void* q, const float* out,
                         const void* workspace, size_t workspace_bytes, bool any_state = true) {
    if (!q || !out || !aligned16(q) || !aligned16(out)) return KIVI_ERR_INVALID_ARG;
    const int length = c->n_kq + c->n_kr;
    if (length < 1 || length != c->n_vq + c->n_vr) return KIVI_ERR_INVALID_ARG;
    size_t need = 0;
    if (any_state) kivi_decode_workspace_bytes(l, &need);
    if (!workspace || !aligned16(workspace) || workspace_bytes < need) return KIVI_ERR_WORKSPACE;
    return KIVI_OK;
}

int decode_family(const kivi_layout_t* l) {
    // the matrix-core family unless the caller asks for the vector ALUs or it has no instantiation
    // for this (bits, query heads per kv-head)
    const int rep = std::min(l->n_q_heads / l->n_kv_heads, kMaxRep);
    if (l->decode_path == KIVI_DECODE_VALU) return KIVI_DECODE_VALU;
    return mfma_geometry(l->bits, rep).chunk_tiles == 0 ? KIVI_DECODE_VALU : KIVI_DECODE_MFMA;
}

// The matrix-core family as two launches (fp16 rows first, then the all-quantised chunks): possible
// when the cache has both parts and K and V are split at the same token; chosen when asked for, or
// by three measured rules.
//  (1) A workgroup of the persistent kernel would own several (batch, kv-head) units: their fp16-row
//      chunks would run one after the other, each a chain of dependent steps (32 heads, context 4096,
//      2 bits: equal at 1 unit per workgroup, 4-6 % faster from 1.5 on).
//  (2) Between half a unit and one unit per workgroup most workgroups straddle two units and run two
//      such chains: two launches are 2-12 % faster once the launch is long enough to carry the
//      second launch's fixed 8-12 us.
// With 3 or more query heads per kv-head (decode_tiles_kernel) the fp16 rows have workgroups of their own in
// one launch, where they take residency from workgroups that run much longer, and ragged_rows_kernel as a launch of their own,
// which costs 4-5 us where nothing is gained.  Whole steps, one launch / two, us:
//  (3) 5 to 8 heads: from 384 fp16-row tiles on.  8 heads, 512 units, 1000 tokens 44.0 / 35.5, 4000 87.8 / 64.8 (4 bits 106.8 / 81.6);
//      384 units, 4000 52.7 / 53.1 (58.9 / 66.8), 256 units 37.6 / 37.8; 128 units 22.8 / 27.8, 1000 tokens 15.6 / 19.7: the line would
//      be better at 512 units now (it was drawn when the fp16 rows were 40 % of a single launch).
//  (4) 3 or 4 heads: 512 units on (1000 tokens 36.9 / 29.9, 4000 76.0 / 57.0, 4 bits 88.7 / 72.2), and 384 with long contexts (4000
//      49.1 / 45.9, 4 bits 53.3 / 57.1; 1000 20.1 / 26.8).
//  (5) Neither for short contexts while the units are fewer than the resident workgroups.  (Drawn when the first launch was
//      decode_tiles_kernel's or residual_rows_kernel's: 512 units, 15 tiles, 3 heads 28.3 / 30.0.  With ragged_rows_kernel two are ahead there:
//      488 tokens, 3 heads 26.3 / 24.4, 8 heads 31.6 / 30.8, with a flush 31.7 / 27.4 and 35.4 / 32.7; 1024 units 45.5 / 39.1 and 54.6 / 45.9.)
// `flush`: the step also flushes and the fp16-row launch could carry that out (G = 32).
//  (0) Two heads: a flush has to end before the launch that reads its tiles, so the single-launch form of decode_mfma_kernel takes
//      two launches as well, the first of them nearly empty: then it rides with the fp16 rows at no cost of its own.  Up to 384
//      units and units x tiles of 40 000 decode_tiles_kernel carries it in its only launch (136 units x 8191 tokens 41.2 -> 35.0 us, 192 x
//      4095 32.7 -> 26.7, 256 x 4095 35.2 -> 34.2, 384 x 2047 35.4 -> 30.4; beyond: 384 x 4095 48.3 / 49.8, 256 x 16 383 91.2 / 96.8).
// One head: decode_one_kernel, a single launch unless the caller asks for two (one_launch); (1) and (2) only decide the plan's
// pieces, and with them the workspace that the call asks for.
constexpr int kTwoHeadTilesUnits = 384;
bool wants_two_launches(const kivi_layout_t* l, const kivi_cache_t* c, int path, bool flush = false) {
    if (path != KIVI_DECODE_MFMA || l->decode_path == KIVI_DECODE_MFMA_ONE) return false;
    const int rep_launch = std::min(l->n_q_heads / l->n_kv_heads, kMaxRep);
    const int rep_variant = rep_launch <= 2 ? rep_launch : (rep_launch <= 4 ? 4 : 8);
    const int tiles_total = ceil_div(c->n_kq + c->n_kr, kTileTokens);
    const int tiles_b = tiles_total - c->n_kq / kTileTokens;
    const bool possible = c->n_kq == c->n_vq && c->n_kq >= kTileTokens && c->n_kr > 0 &&
                          residual_rows_possible(tiles_b, rep_variant);
    if (!possible) return false;
    if (l->decode_path == KIVI_DECODE_MFMA_TWO) return true;
    const int64_t units = (int64_t)l->batch * l->n_kv_heads;
    const int64_t work = units * tiles_total, row_work = units * tiles_b;
    if (flush && rep_variant == 2 && units > 128) return units > kTwoHeadTilesUnits || work > 40000; // (0)
    if (rep_variant >= 4 && units < 768 && tiles_total <= 20) return false;                          // (5)
    if (rep_variant == 8) return tiles_b >= 2 && work >= 4000 && row_work >= 384;                    // (3)
    if (rep_variant == 4) return units >= 512 || (units >= 384 && work >= 40000);                    // (4)
    const int resident = mfma_geometry(l->bits, rep_launch).resident_workgroups;
    if (units * 4 >= (int64_t)resident * 5) return true;                                             // (1)
    return units * 2 > resident && units < resident && tiles_b >= 2 && work >= 24000;                // (2)
}

// With 4, 6 or 8 query heads per kv-head and less work than the chip has room for, equal parts of every group run
// as units of their own (the instantiation for a part's heads needs fewer instructions per tile, and the cache is read
// once per part, which such launches do not notice).  Limit: one chunk per resident workgroup -- from there on the
// doubled number of tiles costs more (64 query / 8 kv heads, batch 4, context 16384: 48 us in halves, 31 us whole).
// log2 of the parts a kv-head's query heads are served in: 0 (whole group), 1 (halves), 2 (quarters)
int head_split_shift(const kivi_layout_t* l, const SplitPlan& plan, int path, bool two_launches) {
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    if (path != KIVI_DECODE_MFMA || two_launches || (rep_total != 4 && rep_total != 6 && rep_total != 8)) return 0;
    if (l->group != kTileTokens) return 0;
    const int64_t units = (int64_t)l->batch * l->n_kv_heads, chunks = units * plan.n_splits();
    // parts of 2 heads: 2 bits only, where these limits were measured (the comparison is of the chunks that plans are
    // reported in; decode_tiles_kernel cuts its work itself)
    const MfmaGeometry g2 = mfma_geometry(l->bits, 2);
    const bool two_heads_possible = g2.chunk_tiles == plan.tiles_per_split_a;
    if (rep_total == 8 && two_heads_possible && units <= 16 && chunks <= g2.resident_workgroups) return 2;     // quarters
    if (rep_total == 4)     // 2 + 2: up to 64 units
        return two_heads_possible && units <= 64 && chunks <= g2.resident_workgroups ? 1 : 0;
    return chunks <= mfma_geometry(l->bits, 4).resident_workgroups ? 1 : 0;
}

// A group wider than kMaxRep heads is served as runs of kWideGroupRun query heads in ONE launch of the single-launch
// form (1: the group fits one pass, or the form is not the single launch: then one launch, or pair, per kMaxRep
// heads).  decode_tiles_kernel takes two neighbouring runs in one pass over the cache: its eight head slots cost a
// tile 15 % more than four.
constexpr int kWideGroupRun = 4;
int wide_group_runs(const kivi_layout_t* l, int path, bool two_launches) {
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    if (path != KIVI_DECODE_MFMA || two_launches || rep_total <= kMaxRep) return 1;
    return ceil_div(rep_total, kWideGroupRun);
}

// Which kernel of the matrix-core family serves the layout: decode_tiles_kernel from three query heads per
// kv-head on (sweeps over 8-1024 units, contexts 200-30 000, 2 and 4 bits, G = 32 to 128, both policies: 1.0-2.7 times as
// fast as decode_mfma_kernel was, but 0.88-0.97 at 512 units with K and V split differently, mostly with 4 heads, before the rows had
// a launch there), and with two heads up to 384 units where that is one
// launch (320 units x 2047 tokens with a flush 35.1 -> 28.9 us, 384 x 1000 28.8 -> 20.0, split differently 288 x 2000 35.0 -> 28.1; from
// 512 units on that kernel's cheaper tiles win: 512 x 1000 28.4 / 29.5 us, 4 bits, 512 x 4000 69.0 / 77.3).  With one head per kv-head most of its matrix columns would idle.
bool uses_tiles(const kivi_layout_t* l, const kivi_cache_t* c) {
    const int rep = l->n_q_heads / l->n_kv_heads;
    if (rep != 2) return rep >= 3;
    // (K and V split differently, 384 units x 8000 tokens: 88.9 us here, 81.1 there; x 4000, 4 bits 59.0 / 65.7)
    const int64_t units = (int64_t)l->batch * l->n_kv_heads, work = units * ceil_div(c->n_kq + c->n_kr, kTileTokens);
    return (units <= 256 || (units <= kTwoHeadTilesUnits && work <= 64000)) && l->decode_path != KIVI_DECODE_MFMA_TWO;
}
// K and V split at different tokens (Algorithm 1's policy), decode_tiles_kernel: the tiles that are not all quantised in a
// launch of their own, as in the two-launch form, where they would take the residency of the others in one.  From 512 units
// on and not for short contexts (one launch / two, 1500 tokens, 4 heads, 512 and 1024 units 52.3 / 45.1, 88.3 / 78.6 us; 8 heads, 512 units
// 55.2 / 51.0; 500 tokens, 4 heads 34.2 / 36.4 and 56.0 / 58.9; 384 units, 1500 tokens 28.1 / 41.7).
bool rows_launch_for_uneven_split(const kivi_layout_t* l, const kivi_cache_t* c, int path) {
    return path == KIVI_DECODE_MFMA && l->decode_path != KIVI_DECODE_MFMA_ONE && uses_tiles(l, c) && l->n_q_heads <= kMaxRep * l->n_kv_heads &&
           c->n_kq != c->n_vq && std::min(c->n_kq, c->n_vq) >= kTileTokens && (int64_t)l->batch * l->n_kv_heads >= 512 &&
           ceil_div(c->n_kq + c->n_kr, kTileTokens) > 20;
}

// One query head per kv-head and no value token quantised before its key: decode_one_kernel, a single launch (unless the caller
// asks for two), whatever wants_two_launches says; the plan's pieces are its need of workspace then.
bool one_launch(const kivi_layout_t* l, const kivi_cache_t* c, int path) {
    return path == KIVI_DECODE_MFMA && l->decode_path != KIVI_DECODE_MFMA_TWO && l->n_q_heads == l->n_kv_heads && c->n_kq >= c->n_vq;
}

// Launches of one attention call: a group wider than kMaxRep heads takes one pass per kMaxRep heads, except in the
// matrix-core family's single-launch form, where the runs are units of one launch.
int attention_launches(const kivi_layout_t* l, const kivi_cache_t* c, int path, bool two_launches) {
    if (one_launch(l, c, path)) return 1;
    if (rows_launch_for_uneven_split(l, c, path)) return 2;
    const int passes = wide_group_runs(l, path, two_launches) > 1 ? 1 : ceil_div(l->n_q_heads / l->n_kv_heads, kMaxRep);
    return path == KIVI_DECODE_MFMA ? (two_launches ? 2 : 1) * passes : passes + 1;      // vector-ALU family: decodes + merge
}

// parts per (batch, query head) that `bytes` of workspace have room for
int part_rows(const kivi_layout_t* l, size_t bytes) {
    const size_t row = (size_t)l->batch * l->n_q_heads * (kHeadDim + 2) * sizeof(float);
    const int n = (int)std::min<size_t>(bytes / row, kTilesMaxParts);
    return n > 1 ? n & ~1 : n;      // even: the statistics of a row's first part are 16-byte aligned
}

// Launch the attention of q over cache state `c` (already validated).  k_new / v_new non-null: the
// rows of token length-1 are not in the rings yet and the (matrix-core) kernel puts them there.
// flush_k / flush_v non-null (two-launch form, decode_tiles_kernel, or one query head per kv-head): the residual flush that produced
// state `c` has not been launched yet.  A single launch quantises the tokens itself, of two the first with extra workgroups.
int enqueue_attention(const kivi_layout_t* l, const kivi_cache_t* c, const void* q, float softmax_scale,
                      float* out, void* workspace, size_t workspace_bytes, const void* k_new, const void* v_new,
                      void* stream, const QuantKeyParams* flush_k = nullptr, const QuantValueParams* flush_v = nullptr) {
    const int length = c->n_kq + c->n_kr;
    DecodeParams p{};
    p.k_codes = static_cast<const uint32_t*>(c->k_codes);
    p.k_scale = static_cast<const __half*>(c->k_scale);
    p.k_zero = static_cast<const __half*>(c->k_zero);
    p.v_codes = static_cast<const uint32_t*>(c->v_codes);
    p.v_scale = static_cast<const __half*>(c->v_scale);
    p.v_zero = static_cast<const __half*>(c->v_zero);
    p.k_resid = static_cast<const __half*>(c->k_resid);
    p.v_resid = static_cast<const __half*>(c->v_resid);
    p.n_kq = c->n_kq; p.n_vq = c->n_vq; p.k_r_start = c->k_r_start; p.n_kr = c->n_kr;
    p.v_r_start = c->v_r_start; p.n_vr = c->n_vr;
    p.cap_tiles = l->cap_q_tokens / kTileTokens; p.cap_r = l->cap_r_tokens;
    p.q = static_cast<const __half*>(q); p.out = out;
    p.softmax_scale = softmax_scale;
    p.batch = l->batch; p.n_q_heads = l->n_q_heads; p.n_kv_heads = l->n_kv_heads; p.bits = l->bits;
    p.kg_shift = l->group == 32 ? 0 : (l->group == 64 ? 1 : 2);
    p.length = length;
    const int path = decode_family(l);
    if ((k_new || v_new) && path != KIVI_DECODE_MFMA) return KIVI_ERR_UNSUPPORTED;
    p.k_new = static_cast<const __half*>(k_new); p.v_new = static_cast<const __half*>(v_new);
    const bool two = wants_two_launches(l, c, path, flush_k || flush_v);
    p.plan = plan_splits(l, c, path == KIVI_DECODE_MFMA, two);
    p.two_launches = two ? 1 : 0;
    p.head_groups = wide_group_runs(l, path, two);
    const bool one = one_launch(l, c, path);
    const bool tiles = path == KIVI_DECODE_MFMA && uses_tiles(l, c) && !(two && l->n_q_heads <= 2 * l->n_kv_heads);
    if ((flush_k || flush_v) && !one && !((two || tiles) && flush_k && flush_v)) return KIVI_ERR_INVALID_ARG;
    p.flush_k = flush_k;
    p.flush_v = flush_v;
    const size_t rows = (size_t)l->batch * l->n_q_heads * p.plan.n_splits();
    if (counter_bytes(l) + rows * (kHeadDim + 2) * sizeof(float) > workspace_bytes) return KIVI_ERR_WORKSPACE;
    p.counters = static_cast<int32_t*>(workspace);
    if (tiles && rows_launch_for_uneven_split(l, c, path)) p.two_launches = 1;
    p.part_stride = p.plan.n_splits();
    if (tiles || one) p.part_stride = part_rows(l, workspace_bytes - counter_bytes(l));
    p.part_o = reinterpret_cast<float*>(static_cast<char*>(workspace) + counter_bytes(l));
    p.part_ml = p.part_o + (size_t)l->batch * l->n_q_heads * p.part_stride * kHeadDim;

    hipStream_t hs = static_cast<hipStream_t>(stream);
    // Up to kMaxRep query heads per kv-head go through one launch.  A wider group (multi-query
    // attention: 71 heads on one kv-head) takes one launch per kMaxRep heads, each reading the cache
    // again; the launches share the plan and the workspace (their part rows are disjoint, and the
    // matrix-core kernel leaves its counters at zero).  Only the first one appends the new token.
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    p.rep_variant = std::min(rep_total, kMaxRep);
    if (p.head_groups > 1) {
        // a group wider than kMaxRep heads in the single-launch form: its runs of kWideGroupRun heads are
        // units of ONE launch (they read the same cache, which the caches serve after the first)
        p.q_head0 = 0;
        p.rep_here = 2 * kWideGroupRun;             // two neighbouring runs share one pass
        p.rep_variant = p.rep_here;
        p.head_groups = ceil_div(rep_total, p.rep_here);
        return hip_status(launch_decode_tiles(p, hs));
    }
    if (one) return hip_status(launch_decode_one(p, hs));
    if (const int shift = head_split_shift(l, p.plan, path, two)) {
        p.head_groups = 1 << shift;
        p.q_head0 = 0;
        p.rep_here = rep_total >> shift;
        p.rep_variant = p.rep_here <= 2 ? 2 : 4;
        return hip_status(launch_decode_tiles(p, hs));
    }
    for (int h0 = 0; h0 < rep_total; h0 += kMaxRep) {
        p.q_head0 = h0;
        p.rep_here = std::min(kMaxRep, rep_total - h0);
        hipError_t e = path != KIVI_DECODE_MFMA ? launch_decode_valu(p, hs) : tiles ? launch_decode_tiles(p, hs) : launch_decode_mfma(p, hs);
        if (e == hipErrorNotSupported) return KIVI_ERR_UNSUPPORTED;
        if (int s = hip_status(e)) return s;
        p.k_new = p.v_new = nullptr;
        p.flush_k = nullptr;
        p.flush_v = nullptr;
    }
    // the matrix-core kernel merges its splits itself; the vector-ALU family uses a second launch
    return path == KIVI_DECODE_MFMA ? KIVI_OK : hip_status(launch_merge(p, hs));
}

}  // namespace

namespace {

inline bool same_state(const kivi_seq_state_t& a, const kivi_seq_state_t& b) {
    return a.n_kq == b.n_kq && a.n_vq == b.n_vq && a.k_r_start == b.k_r_start && a.n_kr == b.n_kr &&
           a.v_r_start == b.v_r_start && a.n_vr == b.n_vr;
}

// Walk the batch in runs of equal state; `call(sub_layout, sub_cache, b0)` handles one run and may
// change the sub-cache's integer fields, which are then written back to the run's states.
template <class F>
int for_each_run(const kivi_layout_t* l, const kivi_cache_t* c, kivi_seq_state_t* states, bool write_back, F&& call) {
    if (int s = check_layout(l)) return s;
    if (!c || !states) return KIVI_ERR_INVALID_ARG;
    for (int b0 = 0; b0 < l->batch;) {
        int b1 = b0 + 1;
        while (b1 < l->batch && same_state(states[b0], states[b1])) ++b1;
        kivi_layout_t sl;
        kivi_cache_t sc;
        if (int s = kivi_batch_slice(l, c, b0, b1 - b0, &states[b0], &sl, &sc)) return s;
        if (int s = call(sl, sc, b0)) return s;
        if (write_back)
            for (int b = b0; b < b1; ++b)
                states[b] = kivi_seq_state_t{sc.n_kq, sc.n_vq, sc.k_r_start, sc.n_kr, sc.v_r_start, sc.n_vr};
        b0 = b1;
    }
    return KIVI_OK;
}

}  // namespace

// ---- batches of different lengths in one pair of launches ----
namespace {

constexpr int kNotApplicable = 1;       // (internal) the fast path does not serve this batch: use the run-by-run path

// Attention over a batch whose sequences differ in length as ONE pair of launches (a pair per 8 heads for 9 to 16 query heads per
// kv-head).  Two heads and more: ragged_rows_kernel has the fp16 rows of every unit, appends the new token when k_new / v_new are
// given and makes the tables by which decode_tiles_kernel cuts the packed tokens of all units evenly.  One head: the first
// launch makes decode_one_kernel's table only (more than kInlineSequences: the host does).  Served: K and V split alike in every
// sequence, at least one fp16 row and as many tiles of them as residual_rows_possible allows, at least one quantised tile somewhere
// in the batch, and with G > 32 more runs than run_by_run takes.
// ragged_plan decides everything that can refuse the batch, on the host and without a launch (a step plans before it
// flushes): `st` are the states the attention sees (after append and flush); kNotApplicable for any other batch.
// ragged_launch then carries the plan out.
struct RaggedPlan {
    DecodeParams p;             // all but the addresses and the query
    bool tiles;                 // decode_tiles_kernel, and launch_ragged_rows before it
    bool tables_on_device;      // ... which makes the tables itself
    bool in_arguments;          // the first launch takes the counters as arguments (otherwise they are copied)
    int max_row_tiles;          // of any sequence
    int units_per_sequence;     // decode_tiles_kernel
    std::vector<OneHeadSequence> sequences;     // decode_one_kernel, longest first
    size_t parts_offset;        // of the parts in the workspace
    // what the kernels read per call, int32: the sequences' counters (state_ints with the padding), the workgroups' table
    // from state_ints on and the sequences' from unit_table on (left to the first launch with tables_on_device); one head per
    // kv-head: the sequences' table, and their first workgroups from unit_table on (left to the first launch with in_arguments)
    std::vector<int32_t> tables;
    size_t state_ints, unit_table;
    std::vector<int32_t> steps;
};

// The second launch: decode_tiles_kernel from two heads per kv-head on, decode_one_kernel for one.  (Two heads, decode_mfma_kernel's forms for
// such batches before, whole steps: 32 units 29.1 -> 25.8 us, 128 of 500-8000 tokens 44.6 -> 28.5, 512 of 2000-2200 43.4 -> 41.5, of
// 500-8000 96 -> 64, 1024 of 500-4000 134 -> 72, 2048 of 1000-1100 89 -> 85; the least gain, none, at 512 of 4000-4200 and 4 bits.)
// One pair of launches for up to 8 heads, a pair per 8 for up to 16, and from 17 on one pair with runs of 8 heads as units of
// their own, as in a batch of one length.
bool ragged_on_tiles(const kivi_layout_t* l) { return l->n_q_heads >= 2 * l->n_kv_heads; }
int ragged_runs(const kivi_layout_t* l) {
    const int rep = l->n_q_heads / l->n_kv_heads;
    return rep > 2 * kMaxRep ? ceil_div(rep, kMaxRep) : 1;
}
// G > 32: few runs of equal sequences take a call of the uniform entry point each.
// All sequences alike: one call where it is faster than the pair (1 sequence of 8000 tokens, G = 64, one call / the pair: 32 / 32 heads 12.0 /
// 15.0 us, 16 / 8 13.0 / 21.3, 64 / 8 18.3 / 29.2; 16 of 4000, 32 / 8 22.9 / 25.8).  The pair's time over the call's, G = 64, 2 bits:
//   units                 128   256   320   384   448   512   640   768  1024  1664  2048
//   2 heads, 1000 tokens 1.50  1.30  1.27  1.36  0.78  1.08  0.96  0.83  0.98  1.09  1.31     (one head at least 1.05 everywhere)
//   2 heads, 4000        1.28  1.06  1.00  0.92        1.02        0.92  0.98
//   4 heads, 300         1.13  1.02  1.01  1.02  0.88  0.88  0.82  0.92  0.91  1.25  1.21
//   4 heads, 1000        1.44  1.27  1.24  1.31  0.89  1.04  1.03  0.97  0.98  1.18  1.15
//   4 heads, 4000        1.24  1.03  0.96  1.02        1.01        0.98  0.99
//   8 heads, 300         1.21  1.08  1.09  1.11  0.86  0.82  0.85  0.95  0.92  1.21  1.18
//   8 heads, 1000        1.59  1.30  1.10  1.12  1.09  1.09  1.05  0.98  1.02  1.17  1.14     (12 heads as 8, up to 2300 units)
// and 12 000 tokens, 256 units: 2 and 4 heads 0.9, 6 heads 1.04.  17 and more heads, a unit per 8: 17 heads, 64 units 1.13-1.58, 128 1.42 at 1000
// tokens, 0.68 at 4000, 192 0.64 at 1000; 32 heads, 96 units 1.41 at 1000, 0.50 at 4000; 71 heads, 32 units 1.05-1.28, 64 0.79-0.87.
bool one_call_for_all(const kivi_layout_t* l, int tokens) {
    const int rep = l->n_q_heads / l->n_kv_heads;
    const int64_t units = (int64_t)l->batch * l->n_kv_heads;
    const bool short_contexts = tokens <= 20 * kTileTokens;             // (line (5) of wants_two_launches)
    if (rep == 1) return true;
    if (ragged_runs(l) > 1) return tokens <= 1024 ? units <= 128 && units * ragged_runs(l) <= 384 : units <= 64 && units * ragged_runs(l) <= 288;
    if (units > 1536) return rep == 2 ? tokens >= 500 : rep <= kMaxRep || units <= 2304;
    if (units <= 384) return rep > 4 || units * tokens <= 1100000;
    return rep > 2 && !short_contexts && units < 768 && (rep > 4 || units >= 512);
}
// From two runs on the pair is the
// faster one (1000 and 3000 tokens, 4 bits, 32 / 8 heads 23.1 / 17.4 us),
// but with 9 to 16 heads it is two pairs against one launch a run.  Two sequences, calls / pairs: 96 / 8 heads, 150-300 tokens 19.7 / 27.7 us,
// 4000-4600 29.3 / 48.7, 12 / 1, 300-1000 22.8 / 32.8, 32 / 2, 9000-10 000 30.7 / 55.4, until the launches are long: two runs, 96 / 8, 64 of
// 300-1000 (10 000 tiles over all kv-heads) 61.6 / 61.5, 32 of 1000-4600 (22 500) 93.8 / 66.1.  Three: 32 / 2, 900-1100 37 / 36; 96 / 8, 2000-2500
// 38.6 / 40.2, 4000-4600 44.5 / 53.2, 32 / 2, 1000-10 000 41.2 / 48.2; but 12 / 1, 8 sequences of 1000-4600 (720 tiles) 39.7 / 37.4 and 160 / 16 (6500) 54.6 / 50.9.
bool run_by_run(const kivi_layout_t* l, const kivi_seq_state_t* st) {
    if (l->group == kTileTokens) return false;
    int runs = 1, longest = 0;
    int64_t tiles = 0;
    for (int b = 0; b < l->batch; ++b) {
        const int tokens = st[b].n_kq + st[b].n_kr;
        if (b > 0 && !same_state(st[b - 1], st[b])) ++runs;
        longest = std::max(longest, tokens);
        tiles += (int64_t)ceil_div(tokens, kTileTokens) * l->n_kv_heads;
    }
    const bool two_pairs = l->n_q_heads > kMaxRep * l->n_kv_heads && ragged_runs(l) == 1;
    if (runs == 1) return one_call_for_all(l, longest);
    return two_pairs && ((runs == 2 && tiles <= 12000) || (runs == 3 && longest > 1500 && tiles >= 800 && tiles <= 5000));
}
int ragged_plan(const kivi_layout_t* l, const kivi_seq_state_t* st, size_t workspace_bytes, RaggedPlan& plan) {
    if (decode_family(l) != KIVI_DECODE_MFMA || l->decode_path == KIVI_DECODE_MFMA_ONE) return kNotApplicable;
    if (l->cap_q_tokens < kTileTokens) return kNotApplicable;
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    const int rep_launch = std::min(rep_total, kMaxRep);
    const int rep_variant = rep_launch <= 2 ? rep_launch : (rep_launch <= 4 ? 4 : 8);
    int max_tiles_a = 0, max_tiles_b = 0;
    for (int b = 0; b < l->batch; ++b) {
        const kivi_seq_state_t& x = st[b];
        if (x.n_kq != x.n_vq || x.n_kr != x.n_vr || x.n_kr < 1 || x.n_kq % kTileTokens != 0) return kNotApplicable;
        const int tiles_a = x.n_kq / kTileTokens;
        max_tiles_a = std::max(max_tiles_a, tiles_a);
        max_tiles_b = std::max(max_tiles_b, ceil_div(x.n_kq + x.n_kr, kTileTokens) - tiles_a);
    }
    if (max_tiles_a < 1 || !residual_rows_possible(max_tiles_b, rep_variant) || run_by_run(l, st)) return kNotApplicable;
    const MfmaGeometry g = mfma_geometry(l->bits, rep_launch);
    if (g.chunk_tiles == 0) return kNotApplicable;
    // (G > 32: with less workspace than documented the batch goes run by run, which asks for no more than each run's)
    size_t documented = 0;
    if (kivi_decode_workspace_bytes(l, &documented) != KIVI_OK || (l->group > kTileTokens && workspace_bytes < documented)) return kNotApplicable;

    DecodeParams& p = plan.p;
    p = DecodeParams{};
    // the scalar counters describe the longest sequence (the kernels take each sequence's own from seq_state)
    p.n_kq = p.n_vq = max_tiles_a * kTileTokens;
    p.n_kr = p.n_vr = max_tiles_b * kTileTokens;
    p.length = p.n_kq + p.n_kr;
    p.cap_tiles = l->cap_q_tokens / kTileTokens; p.cap_r = l->cap_r_tokens;
    p.batch = l->batch; p.n_q_heads = l->n_q_heads; p.n_kv_heads = l->n_kv_heads; p.bits = l->bits;
    p.kg_shift = l->group == 32 ? 0 : (l->group == 64 ? 1 : 2);
    p.plan.tiles_a = max_tiles_a;
    p.plan.tiles_total = max_tiles_a + max_tiles_b;
    p.plan.tiles_per_split_a = g.chunk_tiles;
    p.plan.tiles_per_split_b = max_tiles_b;
    p.plan.n_splits_a = ceil_div(max_tiles_a, g.chunk_tiles);
    p.plan.n_splits_b = 1;
    p.two_launches = 1;
    const size_t parts_offset = plan.parts_offset = counter_bytes(l) + seq_state_bytes(l) + slice_table_bytes(l);
    // up to two heads per kv-head have always asked for room for the longest sequence's splits, also where the plan makes do with less
    const size_t asked = (size_t)l->batch * l->n_q_heads * p.plan.n_splits() * (kHeadDim + 2) * sizeof(float);
    if (rep_total <= 2 && parts_offset + asked > workspace_bytes) return KIVI_ERR_WORKSPACE;

    // What the kernels read per call goes to the device as arguments of the first launch, or (many sequences) in a copy, which is
    // an operation of its own on the stream: the counters, 16 bytes per sequence, out of which the first launch makes the tables, or (one head,
    // room for a single part, more sequences still) the tables too.  (An asynchronous copy out of pageable memory has taken its source
    // when the call returns.)  With the tables copied as well, 250 sequences of 500 tokens, 2 / 1 heads, took 75.7 us in place of 60.8.
    std::vector<int32_t>& tables = plan.tables;
    const bool tiles = plan.tiles = ragged_on_tiles(l);
    plan.in_arguments = plan.tables_on_device = false;
    plan.max_row_tiles = max_tiles_b;
    p.head_groups = tiles ? ragged_runs(l) : 1;
    if (tiles) {
        plan.state_ints = seq_state_bytes(l) / sizeof(int32_t);
        tables.assign(plan.state_ints, 0);
        for (int b = 0; b < l->batch; ++b) {
            const kivi_seq_state_t& x = st[b];
            tables[4 * (size_t)b + 0] = x.n_kq; tables[4 * (size_t)b + 1] = x.n_kr;
            tables[4 * (size_t)b + 2] = x.k_r_start; tables[4 * (size_t)b + 3] = x.v_r_start;
        }
        // the unit-major axis of four-tile steps (at least one per unit) in equal intervals, one per resident workgroup, as far
        // as the units' parts fit (kivi_tiles_plan.h)
        std::vector<int32_t>& steps = plan.steps;
        steps.resize((size_t)l->batch);
        const int units_per_sequence = plan.units_per_sequence = l->n_kv_heads * p.head_groups;
        int64_t all = 0;
        for (int b = 0; b < l->batch; ++b) {
            steps[(size_t)b] = ragged_steps(st[b].n_kq);
            all += (int64_t)steps[(size_t)b] * units_per_sequence;
        }
        if (all > 0x3fffffff) return kNotApplicable;
        const int stride = std::min(part_rows(l, workspace_bytes > parts_offset ? workspace_bytes - parts_offset : 0), tiles_max_parts(l->bits, rep_launch));
        if (stride < 2) return KIVI_ERR_WORKSPACE;
        const int resident = std::min(tiles_resident_ragged(l->bits, rep_launch, l->group > kTileTokens), kMaxSlices);
        RaggedCut cut = ragged_axis(steps, units_per_sequence, resident, stride);
        plan.tables_on_device = l->batch <= kDeviceTableSequences && !cut.whole_units;
        plan.in_arguments = l->batch <= kInlineSequences && plan.tables_on_device;
        if (!plan.tables_on_device) cut = cut_ragged(steps, units_per_sequence, resident, stride, tables);
        p.axis_len = cut.axis.len;
        p.axis_rem = cut.axis.rem;
        plan.unit_table = plan.state_ints + (size_t)cut.workgroups * RaggedCut::kWords;
        p.n_slices = (int32_t)cut.workgroups;
        p.part_stride = stride;
    } else {
        // workgroups in the order of the sequences' lengths: the longest would end last, and alone, otherwise
        std::vector<OneHeadSequence>& sequences = plan.sequences;
        sequences.resize((size_t)l->batch);
        int64_t all = 0;
        for (int b = 0; b < l->batch; ++b) {
            const kivi_seq_state_t& x = st[b];
            const int tiles_a = x.n_kq / kTileTokens;
            const int n = l->bits == 2 ? OneHeadItems<2, false, false>::steps(tiles_a, x.n_kq, x.n_kq, x.n_kr)
                                       : OneHeadItems<4, false, false>::steps(tiles_a, x.n_kq, x.n_kq, x.n_kr);
            sequences[(size_t)b] = OneHeadSequence{0, b, 1, x.n_kq, x.n_kr, x.k_r_start, x.v_r_start, n};
            all += (int64_t)n * l->n_kv_heads;
        }
        std::stable_sort(sequences.begin(), sequences.end(), [](const OneHeadSequence& a, const OneHeadSequence& b) { return a.steps > b.steps; });
        const int stride = std::min(part_rows(l, workspace_bytes > parts_offset ? workspace_bytes - parts_offset : 0), kOneHeadMaxParts);
        if (stride < 1) return KIVI_ERR_WORKSPACE;
        const int cus = one_head_compute_units();
        const int many = l->bits == 2 ? 8 : 12;
        const int near_parts = one_head_near_parts(all, (int64_t)l->batch * l->n_kv_heads, sequences.front().steps, sequences.back().steps, cus, stride, many);
        int64_t wgs = 0;
        for (OneHeadSequence& s : sequences) {
            s.parts = near_parts > 0 ? std::min(near_parts, s.steps) : one_head_ragged_parts(all, s.steps, cus, stride, many);
            s.first_wg = (int32_t)wgs;
            wgs += (int64_t)s.parts * l->n_kv_heads;
            if (wgs > 0x3fffffff) return kNotApplicable;
        }
        p.n_slices = (int32_t)wgs;
        p.part_stride = stride;
        plan.in_arguments = l->batch <= kInlineSequences;
        const size_t entry = sizeof(OneHeadSequence) / sizeof(int32_t);
        plan.state_ints = 0;
        plan.unit_table = (size_t)l->batch * entry;
        tables.resize((size_t)l->batch * (entry + 1));
        if (!plan.in_arguments)
            for (size_t i = 0; i < sequences.size(); ++i) {
                *reinterpret_cast<OneHeadSequence*>(tables.data() + entry * i) = sequences[i];
                tables[plan.unit_table + i] = sequences[i].first_wg;
            }
    }
    const size_t rows = (size_t)l->batch * l->n_q_heads * p.part_stride;
    if (parts_offset + rows * (kHeadDim + 2) * sizeof(float) > workspace_bytes) return KIVI_ERR_WORKSPACE;
    p.rep_variant = rep_launch;
    return KIVI_OK;
}

// flush: the n_flush sequences whose last quantised tile is still in the rings (only with plan.in_arguments).
int ragged_launch(const kivi_layout_t* l, const kivi_cache_t* c, const RaggedPlan& plan, const void* q, float softmax_scale, float* out,
                  void* workspace, const void* k_new, const void* v_new, void* stream, const uint8_t* flush = nullptr, int n_flush = 0) {
    DecodeParams p = plan.p;
    p.k_codes = static_cast<const uint32_t*>(c->k_codes);
    p.k_scale = static_cast<const __half*>(c->k_scale);
    p.k_zero = static_cast<const __half*>(c->k_zero);
    p.v_codes = static_cast<const uint32_t*>(c->v_codes);
    p.v_scale = static_cast<const __half*>(c->v_scale);
    p.v_zero = static_cast<const __half*>(c->v_zero);
    p.k_resid = static_cast<const __half*>(c->k_resid);
    p.v_resid = static_cast<const __half*>(c->v_resid);
    p.k_new = static_cast<const __half*>(k_new); p.v_new = static_cast<const __half*>(v_new);
    p.q = static_cast<const __half*>(q); p.out = out;
    p.softmax_scale = softmax_scale;
    char* ws = static_cast<char*>(workspace);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    int32_t* dev_state = reinterpret_cast<int32_t*>(ws + counter_bytes(l));
    p.counters = reinterpret_cast<int32_t*>(ws);
    if (plan.tiles) p.seq_state = dev_state;
    p.wave_desc = dev_state + plan.state_ints;
    p.unit_parts = dev_state + plan.unit_table;
    p.part_o = reinterpret_cast<float*>(ws + plan.parts_offset);
    p.part_ml = p.part_o + (size_t)l->batch * l->n_q_heads * p.part_stride * kHeadDim;
    // In pieces: up to 16 KB a copy is a kernel of 2 us; for more the stream waits for the copy engine, 13 us longer.
    constexpr size_t kPiece = 16384;
    const size_t copied = plan.in_arguments ? 0 : plan.tables.size() * sizeof(int32_t);
    for (size_t at = 0; at < copied; at += kPiece)
        if (hipMemcpyAsync(reinterpret_cast<char*>(dev_state) + at, reinterpret_cast<const char*>(plan.tables.data()) + at, std::min(kPiece, copied - at),
                           hipMemcpyHostToDevice, hs) != hipSuccess)
            return KIVI_ERR_HIP;
    if (!plan.tiles) {
        const RaggedTables tables{nullptr, nullptr, nullptr, 0, 0, 0, 0, dev_state, dev_state + plan.unit_table};
        if (plan.in_arguments) {
            uint8_t places[kInlineSequences];           // of the sequences that flush, in the table's order
            int n = 0;
            for (size_t i = 0; i < plan.sequences.size(); ++i)
                if (std::find(flush, flush + n_flush, plan.sequences[i].sequence) != flush + n_flush) places[n++] = (uint8_t)i;
            if (int s = hip_status(launch_ragged_one_head(p, plan.sequences.data(), places, n, tables, hs))) return s;
        }
        return hip_status(launch_decode_one(p, hs));
    }
    const RaggedTables device_tables{dev_state, dev_state + plan.unit_table, dev_state + plan.state_ints, p.n_slices, p.axis_len, p.axis_rem,
                                     plan.units_per_sequence, nullptr, nullptr};
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    for (int h0 = 0; h0 < rep_total; h0 += p.head_groups > 1 ? rep_total : kMaxRep) {
        p.q_head0 = h0;
        p.rep_here = std::min(kMaxRep, rep_total - h0);
        DecodeParams rows = p;
        if (p.head_groups > 1) rows.rep_here = rep_total;
        hipError_t e = launch_ragged_rows(rows, plan.max_row_tiles, plan.in_arguments ? plan.tables.data() : nullptr, flush, h0 == 0 ? n_flush : 0,
                                          plan.tables_on_device ? &device_tables : nullptr, hs);
        p.k_new = p.v_new = nullptr;
        if (e == hipSuccess) e = launch_decode_tiles(p, hs);
        if (e == hipErrorNotSupported) return KIVI_ERR_UNSUPPORTED;
        if (int s2 = hip_status(e)) return s2;
    }
    return KIVI_OK;
}

// the calling thread's plan (its tables keep their memory from call to call)
RaggedPlan& thread_plan() {
    static thread_local RaggedPlan plan;
    return plan;
}

// One decoding step of every sequence of a batch of different lengths in one pair of attention
// launches.  A flush of one tile rides in the first of them (G = 32, up to kInlineSequences sequences); any other takes a launch per run of
// equal sequences that flush in this step, which is every G-th step of a sequence.  Served when every sequence's flush leaves the new token in
// the window (then the flush can run out of the rings before the attention appends the token) and
// ragged_plan takes the states after the step.  Returns kNotApplicable with nothing launched and nothing changed
// otherwise.
int ragged_step_fast(const kivi_layout_t* l, const kivi_cache_t* c, kivi_seq_state_t* states, const void* k_new,
                     const void* v_new, const void* q, float softmax_scale, int32_t policy, float* out,
                     void* workspace, size_t workspace_bytes, void* stream) {
    if (check_layout(l) != KIVI_OK || !c || !states) return kNotApplicable;        // the run-by-run path reports the error
    if (policy != KIVI_FLUSH_WINDOW && policy != KIVI_FLUSH_ALG1) return kNotApplicable;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(q) || !aligned16(out) || !workspace || !aligned16(workspace))
        return kNotApplicable;
    if (decode_family(l) != KIVI_DECODE_MFMA || l->batch > 4096) return kNotApplicable;
    // pass 1 (host only): every sequence's flush and its state after the step
    kivi_seq_state_t after[4096];
    int16_t nks[4096], nvs[4096];
    for (int b = 0; b < l->batch; ++b) {
        kivi_layout_t sl; kivi_cache_t sc;
        if (kivi_batch_slice(l, c, b, 1, &states[b], &sl, &sc) != KIVI_OK) return kNotApplicable;
        if (sc.n_kr >= l->cap_r_tokens || sc.n_vr >= l->cap_r_tokens) return kNotApplicable;
        kivi_cache_t ap = sc;
        ap.n_kr += 1; ap.n_vr += 1;
        int nk = 0, nv = 0;
        if (plan_flush(&sl, &ap, policy, &nk, &nv) != KIVI_OK) return kNotApplicable;
        if (nk > sc.n_kr || nv > sc.n_vr || nk > 32767 || nv > 32767) return kNotApplicable;
        nks[b] = (int16_t)nk; nvs[b] = (int16_t)nv;
        after[b] = kivi_seq_state_t{sc.n_kq + nk, sc.n_vq + nv, (sc.k_r_start + nk) % l->cap_r_tokens, sc.n_kr - nk + 1,
                                    (sc.v_r_start + nv) % l->cap_r_tokens, sc.n_vr - nv + 1};
    }
    // the attention's plan: everything that can refuse the step is known before anything is launched
    RaggedPlan& plan = thread_plan();
    if (int s = ragged_plan(l, after, workspace_bytes, plan)) return s;
    // (a step has always asked for room for the longest sequence's splits, also where the plan makes do with less)
    const size_t rows = (size_t)l->batch * l->n_q_heads * (ceil_div(plan.p.plan.tiles_a, plan.p.plan.tiles_per_split_a) + 1);
    if (plan.parts_offset + rows * (kHeadDim + 2) * sizeof(float) > workspace_bytes) return KIVI_ERR_WORKSPACE;
    // pass 2: the flushes.  One tile of a sequence (G = 32), which is what every flush after the first is, rides with the fp16 rows
    // where those have the counters as arguments; others take a launch per run of consecutive sequences with equal state.
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const bool ride = plan.in_arguments && l->group == kTileTokens;
    uint8_t riding[kInlineSequences];
    int n_riding = 0;
    for (int b0 = 0; b0 < l->batch;) {
        int b1 = b0 + 1;
        while (b1 < l->batch && same_state(states[b0], states[b1])) ++b1;
        if (ride && nks[b0] == kTileTokens && nvs[b0] == kTileTokens) {
            for (int b = b0; b < b1; ++b) riding[n_riding++] = (uint8_t)b;
        } else if (nks[b0] > 0 || nvs[b0] > 0) {
            kivi_layout_t sl; kivi_cache_t sc;
            if (int s = kivi_batch_slice(l, c, b0, b1 - b0, &states[b0], &sl, &sc)) return s;
            if (int s = enqueue_flush(&sl, &sc, nks[b0], nvs[b0], hs)) return s;
        }
        b0 = b1;
    }
    if (int s = ragged_launch(l, c, plan, q, softmax_scale, out, workspace, k_new, v_new, stream, riding, n_riding)) return s;
    for (int b = 0; b < l->batch; ++b) states[b] = after[b];
    return KIVI_OK;
}

}  // namespace

// ---- kivi_decode_attention_static: the attention workspace as an array inside the library ----
// For callers that cannot allocate.  Every device the library runs on holds its own copy of the
// array at its own address; in host code the array's name is only a handle for
// hipGetSymbolAddress, the kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[KIVI_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kMaxScratchDevices = 64;
std::atomic<void*> scratch_ptr[kMaxScratchDevices];

// Address of `scratch` on the current device: resolved once per device (with that device
// current), kept afterwards.
int static_scratch_address(void** out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return KIVI_ERR_HIP;
    if (dev < 0 || dev >= kMaxScratchDevices) return KIVI_ERR_UNSUPPORTED;
    void* ptr = scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return KIVI_ERR_HIP;
        scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return KIVI_OK;
}

__global__ void zero_words_kernel(uint32_t* dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0u;
}

}  // namespace

extern "C" {

const char* kivi_status_string(int status) {
    switch (status) {
        case KIVI_OK: return "KIVI_OK";
        case KIVI_ERR_INVALID_ARG: return "KIVI_ERR_INVALID_ARG";
        case KIVI_ERR_UNSUPPORTED: return "KIVI_ERR_UNSUPPORTED";
        case KIVI_ERR_WORKSPACE: return "KIVI_ERR_WORKSPACE";
        case KIVI_ERR_HIP: return "KIVI_ERR_HIP";
        default: return "KIVI_ERR_UNKNOWN";
    }
}

int kivi_cache_sizes(const kivi_layout_t* l, kivi_cache_sizes_t* out) {
    if (int st = check_layout(l)) return st;
    if (!out) return KIVI_ERR_INVALID_ARG;
    const size_t units = (size_t)l->batch * l->n_kv_heads;
    const size_t tiles = (size_t)l->cap_q_tokens / kTileTokens;
    const size_t words = (size_t)kTileTokens * kHeadDim * l->bits / 32;
    out->k_codes = out->v_codes = units * tiles * words * 4;
    // one scale / zero-point per group: keys per (G tokens, channel), values per (token, G channels)
    out->k_scale = out->k_zero = units * ((size_t)l->cap_q_tokens / l->group) * kHeadDim * 2;
    out->v_scale = out->v_zero = units * (size_t)l->cap_q_tokens * (kHeadDim / l->group) * 2;
    out->k_resid = out->v_resid = units * (size_t)l->cap_r_tokens * kHeadDim * 2;
    return KIVI_OK;
}

int kivi_decode_plan(const kivi_layout_t* l, const kivi_cache_t* c, kivi_decode_plan_t* out) {
    if (int st = check_layout(l)) return st;
    if (int st = check_cache(l, c)) return st;
    if (!out) return KIVI_ERR_INVALID_ARG;
    const int path = decode_family(l);
    const bool two = wants_two_launches(l, c, path);
    const SplitPlan plan = plan_splits(l, c, path == KIVI_DECODE_MFMA, two);
    out->family = path;
    const int runs = wide_group_runs(l, path, two);
    out->launches = attention_launches(l, c, path, two);
    out->units_per_kv_head = runs > 1 ? runs : 1 << head_split_shift(l, plan, path, two);
    out->splits_quantised = plan.n_splits_a;
    out->splits_fp16 = plan.n_splits_b;
    out->tiles_per_split_quantised = plan.tiles_per_split_a;
    out->tiles_per_split_fp16 = plan.tiles_per_split_b;
    return KIVI_OK;
}

int kivi_decode_workspace_bytes(const kivi_layout_t* l, size_t* bytes) {
    if (int st = check_layout(l)) return st;
    if (!bytes) return KIVI_ERR_INVALID_ARG;
    const size_t rows = (size_t)l->batch * l->n_q_heads * max_splits(l);
    *bytes = counter_bytes(l) + seq_state_bytes(l) + slice_table_bytes(l) + rows * (kHeadDim + 2) * sizeof(float);
    return KIVI_OK;
}

int kivi_quantize_key_groups(const kivi_layout_t* l, const void* k, int64_t sb, int64_t sh, int64_t st,
                             int32_t n_tokens, kivi_cache_t* c, void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (int s = check_source(k, sb, sh, st)) return s;
    if (n_tokens < 0 || n_tokens % l->group != 0) return KIVI_ERR_INVALID_ARG;
    if ((int64_t)c->n_kq + n_tokens > l->cap_q_tokens) return KIVI_ERR_INVALID_ARG;
    if (n_tokens == 0) return KIVI_OK;
    const RowSource src{static_cast<const __half*>(k), sb, sh, st, 0, 0};
    if (int s = enqueue_key_quant(l, c, src, n_tokens, static_cast<hipStream_t>(stream))) return s;
    c->n_kq += n_tokens;
    return KIVI_OK;
}

int kivi_quantize_value_tokens(const kivi_layout_t* l, const void* v, int64_t sb, int64_t sh, int64_t st,
                               int32_t n_tokens, kivi_cache_t* c, void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (int s = check_source(v, sb, sh, st)) return s;
    if (n_tokens < 0) return KIVI_ERR_INVALID_ARG;
    if ((int64_t)c->n_vq + n_tokens > l->cap_q_tokens) return KIVI_ERR_INVALID_ARG;
    if (n_tokens == 0) return KIVI_OK;
    const RowSource src{static_cast<const __half*>(v), sb, sh, st, 0, 0};
    if (int s = enqueue_value_quant(l, c, src, n_tokens, static_cast<hipStream_t>(stream))) return s;
    c->n_vq += n_tokens;
    return KIVI_OK;
}

int kivi_append_residual(const kivi_layout_t* l, kivi_cache_t* c, const void* k_new, const void* v_new,
                         void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (!k_new || !v_new || !aligned16(k_new) || !aligned16(v_new)) return KIVI_ERR_INVALID_ARG;
    if (c->n_kr >= l->cap_r_tokens || c->n_vr >= l->cap_r_tokens) return KIVI_ERR_INVALID_ARG;
    const int64_t sh = kHeadDim, sb = sh * l->n_kv_heads;
    CopyRowsParams p{};
    p.cap_r = l->cap_r_tokens; p.n_kv_heads = l->n_kv_heads; p.batch = l->batch;
    p.job[0] = {static_cast<const __half*>(k_new), sb, sh, kHeadDim, 0, static_cast<__half*>(c->k_resid),
                (c->k_r_start + c->n_kr) % l->cap_r_tokens, 1};
    p.job[1] = {static_cast<const __half*>(v_new), sb, sh, kHeadDim, 0, static_cast<__half*>(c->v_resid),
                (c->v_r_start + c->n_vr) % l->cap_r_tokens, 1};
    if (int s = hip_status(launch_copy_rows(p, static_cast<hipStream_t>(stream)))) return s;
    c->n_kr += 1;
    c->n_vr += 1;
    return KIVI_OK;
}

int kivi_flush_residual(const kivi_layout_t* l, kivi_cache_t* c, int32_t policy, int32_t* n_key_flushed,
                        int32_t* n_value_flushed, void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (policy != KIVI_FLUSH_WINDOW && policy != KIVI_FLUSH_ALG1) return KIVI_ERR_INVALID_ARG;
    int nk = 0, nv = 0;
    if (int s = plan_flush(l, c, policy, &nk, &nv)) return s;
    if (int s = enqueue_flush(l, c, nk, nv, static_cast<hipStream_t>(stream))) return s;
    if (n_key_flushed) *n_key_flushed = nk;
    if (n_value_flushed) *n_value_flushed = nv;
    return KIVI_OK;
}

int kivi_prefill(const kivi_layout_t* l, const void* k, int64_t ksb, int64_t ksh, int64_t kst, const void* v,
                 int64_t vsb, int64_t vsh, int64_t vst, int32_t n_tokens, int32_t policy, kivi_cache_t* c,
                 void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (int s = check_source(k, ksb, ksh, kst)) return s;
    if (int s = check_source(v, vsb, vsh, vst)) return s;
    if (policy != KIVI_FLUSH_WINDOW && policy != KIVI_FLUSH_ALG1) return KIVI_ERR_INVALID_ARG;
    if (n_tokens < 0 || c->n_kq || c->n_vq || c->n_kr || c->n_vr) return KIVI_ERR_INVALID_ARG;
    const int G = l->group, R = l->residual;
    int nkq, nvq;
    if (policy == KIVI_FLUSH_WINDOW) {
        nkq = nvq = std::max(n_tokens - R, 0) / G * G;
    } else {
        nkq = R > 0 ? n_tokens - n_tokens % R : n_tokens / G * G;   // KeyQuant: r = l % R
        nvq = std::max(n_tokens - R, 0);                            // X_Vg = X_V[:l - R]
    }
    const int nkr = n_tokens - nkq, nvr = n_tokens - nvq;
    if (nkq > l->cap_q_tokens || nvq > l->cap_q_tokens || nkr > l->cap_r_tokens || nvr > l->cap_r_tokens)
        return KIVI_ERR_INVALID_ARG;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const RowSource ksrc{static_cast<const __half*>(k), ksb, ksh, kst, 0, 0};
    const RowSource vsrc{static_cast<const __half*>(v), vsb, vsh, vst, 0, 0};
    CopyRowsParams p{};
    p.cap_r = l->cap_r_tokens; p.n_kv_heads = l->n_kv_heads; p.batch = l->batch;
    p.job[0] = {static_cast<const __half*>(k), ksb, ksh, kst, nkq, static_cast<__half*>(c->k_resid), 0, nkr};
    p.job[1] = {static_cast<const __half*>(v), vsb, vsh, vst, nvq, static_cast<__half*>(c->v_resid), 0, nvr};
    const QuantKeyParams kp = key_quant_params(l, c, ksrc, nkq);
    const QuantValueParams vp = value_quant_params(l, c, vsrc, nvq);
    if (prefill_possible(kp, vp)) {
        if (int s = hip_status(launch_prefill(kp, vp, p, hs))) return s;
    } else {
        if (nkq > 0) {
            if (int s = enqueue_key_quant(l, c, ksrc, nkq, hs)) return s;
        }
        if (nvq > 0) {
            if (int s = enqueue_value_quant(l, c, vsrc, nvq, hs)) return s;
        }
        if (int s = hip_status(launch_copy_rows(p, hs))) return s;
    }
    c->n_kq = nkq; c->n_vq = nvq; c->n_kr = nkr; c->n_vr = nvr; c->k_r_start = 0; c->v_r_start = 0;
    return KIVI_OK;
}

int kivi_decode_attention(const kivi_layout_t* l, const kivi_cache_t* c, const void* q, float softmax_scale,
                          float* out, void* workspace, size_t workspace_bytes, void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (int s = check_attention_args(l, c, q, out, workspace, workspace_bytes)) return s;
    return enqueue_attention(l, c, q, softmax_scale, out, workspace, workspace_bytes, nullptr, nullptr, stream);
}

int kivi_decode_attention_static(const kivi_layout_t* l, const kivi_cache_t* c, const void* q,
                                 float softmax_scale, float* out, void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    // argument checks first (they need no device); the workspace pointer is not known yet, an aligned
    // dummy stands in for it
    if (int s = check_attention_args(l, c, q, out, reinterpret_cast<const void*>(uintptr_t{256}),
                                     KIVI_STATIC_WORKSPACE_BYTES, false)) return s;
    void* ws = nullptr;
    if (int s = static_scratch_address(&ws)) return s;
    // The array keeps what the last call on this device left.  The parts are written before they are
    // read; the counters at its start must be zero: a completed call leaves them so, a fill kernel
    // (not a memset, so that the call can be captured into a graph) makes sure.
    if (counter_bytes(l) > KIVI_STATIC_WORKSPACE_BYTES) return KIVI_ERR_WORKSPACE;
    const int n_words = (int)(counter_bytes(l) / sizeof(uint32_t));
    zero_words_kernel<<<(n_words + 255) / 256, 256, 0, static_cast<hipStream_t>(stream)>>>(static_cast<uint32_t*>(ws), n_words);
    if (int s = hip_status(hipGetLastError())) return s;
    // enqueue_attention refuses (KIVI_ERR_WORKSPACE, nothing launched) a state whose counters and parts pass the limit
    return enqueue_attention(l, c, q, softmax_scale, out, ws, KIVI_STATIC_WORKSPACE_BYTES, nullptr, nullptr, stream);
}

int kivi_decode_step(const kivi_layout_t* l, kivi_cache_t* c, const void* k_new, const void* v_new, const void* q,
                     float softmax_scale, int32_t policy, float* out, void* workspace, size_t workspace_bytes,
                     void* stream) {
    if (int s = check_layout(l)) return s;
    if (int s = check_cache(l, c)) return s;
    if (!k_new || !v_new || !aligned16(k_new) || !aligned16(v_new)) return KIVI_ERR_INVALID_ARG;
    if (policy != KIVI_FLUSH_WINDOW && policy != KIVI_FLUSH_ALG1) return KIVI_ERR_INVALID_ARG;
    if (c->n_kr >= l->cap_r_tokens || c->n_vr >= l->cap_r_tokens) return KIVI_ERR_INVALID_ARG;
    // the cache as it will be after the append and the flush: everything is checked against it
    // before anything is launched
    kivi_cache_t after = *c;
    after.n_kr += 1;
    after.n_vr += 1;
    int nk = 0, nv = 0;
    if (int s = plan_flush(l, &after, policy, &nk, &nv)) return s;
    {
        kivi_cache_t fl = after;
        fl.n_kq += nk; fl.n_kr -= nk; fl.n_vq += nv; fl.n_vr -= nv;
        if (int s = check_attention_args(l, &fl, q, out, workspace, workspace_bytes)) return s;
    }
    if (decode_family(l) == KIVI_DECODE_MFMA && nk <= c->n_kr && nv <= c->n_vr) {
        // The tokens to flush were all in the rings before this step: quantise them first (one
        // launch, none on the steps without a flush), then let the attention read the new token from
        // k_new / v_new and store it in the rings itself.  The ring slot of the new token and the
        // cache state seen by the attention are the same as with append -> flush -> attention.
        kivi_cache_t flushed = *c;                       // the counters after the flush, nothing launched yet
        if (int s = enqueue_flush(l, &flushed, nk, nv, nullptr, false)) return s;
        after = flushed;
        after.n_kr += 1;
        after.n_vr += 1;
        // In the two-launch form (G = 32) the launch of the fp16 rows quantises the flushed tokens (three and more query heads per
        // kv-head: one tile; two heads: see wants_two_launches).
        // One query head per kv-head: a flush of one tile, which is what every flushing step after the first has, rides in
        // the attention's only launch, and so does one value token (decode_one_kernel, which has both sides' figures).
        // So does one tile in decode_tiles_kernel's single-launch form.
        const bool in_one = one_launch(l, &after, KIVI_DECODE_MFMA);
        const bool one_tile = l->group == kTileTokens && nk == kTileTokens && nv == kTileTokens && after.n_kq == after.n_vq;
        const bool in_tiles = !in_one && one_tile && uses_tiles(l, &after) && !wants_two_launches(l, &after, KIVI_DECODE_MFMA, true);
        const bool one_value = nk == 0 && nv == 1;
        if ((nk > 0 || nv > 0) &&
            (in_one ? one_tile || one_value
                    : in_tiles || (wants_two_launches(l, &after, KIVI_DECODE_MFMA, true) &&
                                   (l->n_q_heads > 2 * l->n_kv_heads ? one_tile : l->group == kTileTokens)))) {
            const int64_t sh = (int64_t)l->cap_r_tokens * kHeadDim, sb = sh * l->n_kv_heads;
            const RowSource ksrc{static_cast<const __half*>(c->k_resid), sb, sh, kHeadDim, c->k_r_start, l->cap_r_tokens};
            const RowSource vsrc{static_cast<const __half*>(c->v_resid), sb, sh, kHeadDim, c->v_r_start, l->cap_r_tokens};
            const QuantKeyParams kp = key_quant_params(l, c, ksrc, nk);
            const QuantValueParams vp = value_quant_params(l, c, vsrc, nv);
            if (int s = enqueue_attention(l, &after, q, softmax_scale, out, workspace, workspace_bytes, k_new, v_new, stream, nk > 0 || !in_one ? &kp : nullptr, &vp))
                return s;
            *c = after;
            return KIVI_OK;
        }
        if (int s = enqueue_flush(l, c, nk, nv, static_cast<hipStream_t>(stream))) return s;
        if (int s = enqueue_attention(l, &after, q, softmax_scale, out, workspace, workspace_bytes, k_new, v_new, stream)) return s;
        *c = after;
        return KIVI_OK;
    }
    // the flush takes the new token itself (Algorithm 1's key flush, or no residual window): append first
    if (int s = kivi_append_residual(l, c, k_new, v_new, stream)) return s;
    if (int s = kivi_flush_residual(l, c, policy, nullptr, nullptr, stream)) return s;
    return enqueue_attention(l, c, q, softmax_scale, out, workspace, workspace_bytes, nullptr, nullptr, stream);
}

int kivi_batch_slice(const kivi_layout_t* l, const kivi_cache_t* c, int32_t b0, int32_t nb,
                     const kivi_seq_state_t* state, kivi_layout_t* sub_layout, kivi_cache_t* sub_cache) {
    if (int s = check_layout(l)) return s;
    if (!c || !sub_layout || !sub_cache || b0 < 0 || nb < 1 || (int64_t)b0 + nb > l->batch) return KIVI_ERR_INVALID_ARG;
    kivi_cache_sizes_t sz;
    if (int s = kivi_cache_sizes(l, &sz)) return s;
    *sub_layout = *l;
    sub_layout->batch = nb;
    *sub_cache = *c;
    // every array is dense [b][h][...]: one sequence takes 1/batch of it
    auto move = [&](void* base, size_t total) -> void* {
        return base ? static_cast<char*>(base) + total / l->batch * b0 : nullptr;
    };
    sub_cache->k_codes = move(c->k_codes, sz.k_codes); sub_cache->k_scale = move(c->k_scale, sz.k_scale);
    sub_cache->k_zero = move(c->k_zero, sz.k_zero);    sub_cache->v_codes = move(c->v_codes, sz.v_codes);
    sub_cache->v_scale = move(c->v_scale, sz.v_scale); sub_cache->v_zero = move(c->v_zero, sz.v_zero);
    sub_cache->k_resid = move(c->k_resid, sz.k_resid); sub_cache->v_resid = move(c->v_resid, sz.v_resid);
    if (state) {
        sub_cache->n_kq = state->n_kq; sub_cache->n_vq = state->n_vq; sub_cache->k_r_start = state->k_r_start;
        sub_cache->n_kr = state->n_kr; sub_cache->v_r_start = state->v_r_start; sub_cache->n_vr = state->n_vr;
    }
    return check_cache(sub_layout, sub_cache);
}

int kivi_decode_step_ragged(const kivi_layout_t* l, const kivi_cache_t* c, kivi_seq_state_t* states,
                            const void* k_new, const void* v_new, const void* q, float softmax_scale,
                            int32_t policy, float* out, void* workspace, size_t workspace_bytes, void* stream) {
    if (!k_new || !v_new || !q || !out) return KIVI_ERR_INVALID_ARG;
    if (int s = ragged_step_fast(l, c, states, k_new, v_new, q, softmax_scale, policy, out, workspace, workspace_bytes, stream);
        s != kNotApplicable)
        return s;
    return for_each_run(l, c, states, true, [&](kivi_layout_t& sl, kivi_cache_t& sc, int b0) {
        const size_t kv_row = (size_t)l->n_kv_heads * kHeadDim, q_row = (size_t)l->n_q_heads * kHeadDim;
        return kivi_decode_step(&sl, &sc, static_cast<const __half*>(k_new) + b0 * kv_row,
                                static_cast<const __half*>(v_new) + b0 * kv_row,
                                static_cast<const __half*>(q) + b0 * q_row, softmax_scale, policy,
                                out + b0 * q_row, workspace, workspace_bytes, stream);
    });
}

int kivi_decode_launches_ragged(const kivi_layout_t* l, const kivi_seq_state_t* states, int32_t* launches) {
    if (int s = check_layout(l)) return s;
    if (!states || !launches) return KIVI_ERR_INVALID_ARG;
    const int path = decode_family(l);
    const int rep_total = l->n_q_heads / l->n_kv_heads;
    const int head_groups = ragged_runs(l) > 1 ? 1 : ceil_div(rep_total, kMaxRep);
    // the conditions of ragged_plan
    bool fast = path == KIVI_DECODE_MFMA && l->decode_path != KIVI_DECODE_MFMA_ONE && l->cap_q_tokens >= kTileTokens;
    int max_tiles_a = 0, max_tiles_b = 0;
    for (int b = 0; b < l->batch; ++b) {
        const kivi_seq_state_t& x = states[b];
        if (x.n_kq < 0 || x.n_vq < 0 || x.n_kr < 0 || x.n_vr < 0 || x.n_kq + x.n_kr != x.n_vq + x.n_vr) return KIVI_ERR_INVALID_ARG;
        if (x.n_kq != x.n_vq || x.n_kr < 1 || x.n_kq % kTileTokens != 0) fast = false;
        max_tiles_a = std::max(max_tiles_a, x.n_kq / kTileTokens);
        max_tiles_b = std::max(max_tiles_b, ceil_div(x.n_kq + x.n_kr, kTileTokens) - x.n_kq / kTileTokens);
    }
    const int rep_launch = std::min(rep_total, kMaxRep);
    if (fast && max_tiles_a >= 1 && residual_rows_possible(max_tiles_b, rep_launch <= 2 ? rep_launch : (rep_launch <= 4 ? 4 : 8)) &&
        !run_by_run(l, states)) {
        *launches = rep_total == 1 && l->batch > kInlineSequences ? 1 : 2 * head_groups;
        return KIVI_OK;
    }
    // run by run
    int total = 0;
    for (int b0 = 0; b0 < l->batch;) {
        int b1 = b0 + 1;
        while (b1 < l->batch && same_state(states[b0], states[b1])) ++b1;
        const kivi_seq_state_t& x = states[b0];
        if (x.n_kq + x.n_kr > 0) {
            kivi_layout_t sl = *l;
            sl.batch = b1 - b0;
            kivi_cache_t sc{};
            sc.n_kq = x.n_kq; sc.n_vq = x.n_vq; sc.n_kr = x.n_kr; sc.n_vr = x.n_vr;
            total += attention_launches(&sl, &sc, path, wants_two_launches(&sl, &sc, path));
        }
        b0 = b1;
    }
    *launches = total;
    return KIVI_OK;
}

int kivi_decode_attention_ragged(const kivi_layout_t* l, const kivi_cache_t* c, const kivi_seq_state_t* states,
                                 const void* q, float softmax_scale, float* out, void* workspace,
                                 size_t workspace_bytes, void* stream) {
    if (!q || !out) return KIVI_ERR_INVALID_ARG;
    if (check_layout(l) == KIVI_OK && c && states && aligned16(q) && aligned16(out) && workspace && aligned16(workspace)) {
        bool ok = true;
        for (int b = 0; b < l->batch && ok; ++b) {
            kivi_layout_t sl; kivi_cache_t sc;
            ok = kivi_batch_slice(l, c, b, 1, &states[b], &sl, &sc) == KIVI_OK;     // validates the sequence's counters
        }
        if (ok) {
            RaggedPlan& plan = thread_plan();
            const int s = ragged_plan(l, states, workspace_bytes, plan);
            if (s == KIVI_OK) return ragged_launch(l, c, plan, q, softmax_scale, out, workspace, nullptr, nullptr, stream);
            if (s != kNotApplicable) return s;
        }
    }
    return for_each_run(l, c, const_cast<kivi_seq_state_t*>(states), false,
                        [&](kivi_layout_t& sl, kivi_cache_t& sc, int b0) {
        if (sc.n_kq + sc.n_kr == 0 && sc.n_vq + sc.n_vr == 0) return (int)KIVI_OK;      // empty slots of the batch
        const size_t q_row = (size_t)l->n_q_heads * kHeadDim;
        return kivi_decode_attention(&sl, &sc, static_cast<const __half*>(q) + b0 * q_row, softmax_scale,
                                     out + b0 * q_row, workspace, workspace_bytes, stream);
    });
}

int kivi_stream_read_probe(const void* src, size_t bytes, void* sink, void* stream) {
    if (!src || !sink || !aligned16(src) || !aligned16(sink) || (bytes & 15)) return KIVI_ERR_INVALID_ARG;
    return hip_status(launch_stream_read(src, bytes, static_cast<uint32_t*>(sink), static_cast<hipStream_t>(stream)));
}

}  // extern "C"
