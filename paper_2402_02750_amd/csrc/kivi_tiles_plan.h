// How decode_tiles_kernel's work is cut among workgroups: arithmetic on the host, without any HIP type, so that
// it can be checked without a device.
//
// A unit is (batch entry, kv-head, run of query heads); its all-quantised tiles are steps of four.  Every workgroup
// that holds some of a unit's steps (or of its fp16 rows) leaves one part per query head in the workspace, which
// has `stride` rows per head, and the kernel merges at most `parts_limit` of them.  Both bounds are kept here: a part
// more than there are rows would be written over the next head's.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#if defined(__HIPCC__)
#define KIVI_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define KIVI_HOST_DEVICE inline
#endif

namespace kivi {

constexpr int kStepTiles = 4;          // tiles per step: one per wavefront of a workgroup

// Division by a number that a launch does not change, for dividends below 2^31: three scalar instructions instead of the
// thirty of an integer division.  (m = 2^32 (2^s - d) / d + 1 with 2^(s-1) < d <= 2^s: n / d = (m n / 2^32 + n) / 2^s.)
struct FastDiv {
    uint32_t mul, shift;
    static FastDiv by(uint32_t d) {
        uint32_t s = 0;
        while ((uint64_t{1} << s) < d) ++s;
        return FastDiv{(uint32_t)(((uint64_t{1} << 32) * ((uint64_t{1} << s) - d)) / d + 1), s};
    }
    KIVI_HOST_DEVICE int of(int n) const { return (int)((uint32_t)((((uint64_t)(uint32_t)n * mul) >> 32) + (uint32_t)n) >> shift); }
};

// An axis of steps in intervals of `len`, the first `rem` of them one step longer.
struct StepAxis {
    int32_t len, rem;
    KIVI_HOST_DEVICE int start(int g) const { return g * len + (g < rem ? g : rem); }
    KIVI_HOST_DEVICE int owner(int pos) const {
        const int cut = rem * (len + 1);
        return pos < cut ? (int)((uint32_t)pos / (uint32_t)(len + 1)) : rem + (int)((uint32_t)(pos - cut) / (uint32_t)len);
    }
    // the same with the divisions by len + 1 and len made ready
    KIVI_HOST_DEVICE int owner(int pos, FastDiv by_longer, FastDiv by_len) const {
        const int cut = rem * (len + 1);
        return pos < cut ? by_longer.of(pos) : rem + by_len.of(pos - cut);
    }
};

// The shortest interval that cuts a unit of n steps into at most max_parts (>= 2) parts: intervals of c steps and more
// cut it into at most (n - 1) / c + 2 (rounded down; the first and the last may hold a single step).
inline int64_t shortest_interval(int64_t n, int max_parts) { return (n - 1) / (max_parts - 1) + 1; }

// Batches of sequences of different lengths: the steps of all units, one unit after the other, in equal intervals,
// one per workgroup.  Row 0 of every head holds what the fp16-row launch left.
struct RaggedCut {
    int64_t workgroups = 0;
    StepAxis axis{1, 0};
    bool whole_units = false;          // room for a single part: every workgroup takes whole units, and the axis is one interval
    // {first unit, first step in it, steps, 0} per workgroup, then the steps before each sequence
    static constexpr int kWords = 4;
};

// Query heads that a workgroup of ragged_rows_kernel takes at once: the matrix instruction's 16 columns, or 8 of them where the
// tiles' outputs (kRowsChunkTiles heads times tiles: 62 KB of LDS) ask for it.
constexpr int kRowsChunkTiles = 120;
inline int rows_chunk_heads(int heads, int tiles) { return std::min(heads, tiles <= 7 ? 16 : 8); }
// fp16 rows in a launch of their own: up to 16 tiles, one wavefront each; 8 with five and more heads.  With one and two heads
// residual_rows_kernel takes them all, from three on ragged_rows_kernel, a unit's heads in one workgroup wherever a batch of one
// length sends them there (8 heads x 8 tiles, 4 x 16).  The line of 64, which was residual_rows_kernel's LDS for eight heads, is kept: a
// window of more than 8 tiles under five and more heads takes the single launch, in a batch of different lengths a call per run.
inline bool residual_rows_possible(int tiles_b, int rep_variant) { return tiles_b >= 1 && tiles_b <= 16 && tiles_b * rep_variant <= 64; }

// a unit's steps, of a sequence with n_q quantised tokens (with none: one empty step)
KIVI_HOST_DEVICE int ragged_steps(int n_q) {
    const int tiles = n_q / 32, steps = (tiles + kStepTiles - 1) / kStepTiles;
    return steps < 1 ? 1 : steps;
}
// The intervals' workgroups and axis (no table): see cut_ragged.
inline RaggedCut ragged_axis(const std::vector<int32_t>& steps, int n_kv_heads, int64_t max_workgroups, int rows) {
    RaggedCut cut;
    const int max_parts = rows - 1;
    int64_t total = 0, max_steps = 1;
    for (const int32_t s : steps) {
        total += (int64_t)s * n_kv_heads;
        max_steps = std::max<int64_t>(max_steps, s);
    }
    const int64_t units = (int64_t)steps.size() * n_kv_heads;
    cut.whole_units = max_parts < 2;
    cut.workgroups = std::min(max_workgroups, cut.whole_units ? units : total);
    // fewer workgroups than parts cannot cut a unit too often; otherwise total / workgroups, rounded DOWN, is the length
    // that counts: the longer intervals come first, so the last units meet the shorter ones only
    if (!cut.whole_units && cut.workgroups > max_parts)
        cut.workgroups = std::max<int64_t>(max_parts, std::min(cut.workgroups, total / shortest_interval(max_steps, max_parts)));
    cut.axis = cut.whole_units ? StepAxis{0x3fffffff, 0} : StepAxis{(int32_t)(total / cut.workgroups), (int32_t)(total % cut.workgroups)};
    return cut;
}
// Interval g of a cut that is not of whole units, from each sequence's steps and the steps before it (units_per_sequence times the
// former, added up): {first unit, first step in it, steps, 0}.
struct RaggedInterval { int32_t unit, first, steps, none; };
KIVI_HOST_DEVICE RaggedInterval ragged_interval(const int32_t* before, const int32_t* steps, int sequences, int units_per_sequence, StepAxis axis, int g) {
    const int start = axis.start(g);
    int lo = 0, hi = sequences;                        // before[lo] <= start < before[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (before[mid] <= start) lo = mid;
        else hi = mid;
    }
    const int into = start - before[lo], unit = into / steps[lo];
    return RaggedInterval{lo * units_per_sequence + unit, into - unit * steps[lo], axis.start(g + 1) - start, 0};
}

// steps[b]: steps of each of the n_kv_heads units of sequence b (at least 1); rows: parts per head that fit, row 0
// included (at least 2).  Appends the table to `out`.
inline RaggedCut cut_ragged(const std::vector<int32_t>& steps, int n_kv_heads, int64_t max_workgroups, int rows, std::vector<int32_t>& out) {
    const RaggedCut cut = ragged_axis(steps, n_kv_heads, max_workgroups, rows);
    const int64_t units = (int64_t)steps.size() * n_kv_heads;

    const size_t base = out.size();
    out.resize(base + (size_t)cut.workgroups * RaggedCut::kWords + steps.size(), 0);
    int32_t* desc = out.data() + base;
    int32_t* before = desc + (size_t)cut.workgroups * RaggedCut::kWords;
    int32_t cum = 0;
    for (size_t b = 0; b < steps.size(); ++b) {
        before[b] = cum;
        cum += steps[b] * n_kv_heads;
    }
    // (a walk without divisions: a step waits for this table)
    const StepAxis whole{(int32_t)(units / cut.workgroups), (int32_t)(units % cut.workgroups)};
    size_t b = 0;
    int32_t unit = 0, head = 0, first = 0;          // where the interval begins; head: of sequence b
    for (int32_t g = 0; g < (int32_t)cut.workgroups; ++g, desc += RaggedCut::kWords) {
        desc[0] = unit;
        desc[1] = first;
        int32_t left = cut.axis.len + (g < cut.axis.rem), length = left;
        if (cut.whole_units) {
            left = length = 0;
            for (int32_t n = whole.len + (g < whole.rem); n > 0; --n, ++unit) {
                length += steps[b];
                if (++head == n_kv_heads) { head = 0; ++b; }
            }
        }
        desc[2] = length;
        for (first += left; b < steps.size() && first >= steps[b]; ++unit) {
            first -= steps[b];
            if (++head == n_kv_heads) { head = 0; ++b; }
        }
    }
    return cut;
}

// A batch of one length: `rows`, the workgroups of the units' fp16 rows, `row_split` per unit, and intervals of the
// all-quantised steps, `intervals` in all: `unit_wgs` per unit of its own steps, or (0) of all units' steps.
struct UniformCut {
    int row_split = 1, row_wgs = 0, unit_wgs = 0;
    StepAxis axis{1, 0};
    int64_t intervals = 0;
};

// Fewest steps of a workgroup where there are workgroups enough for less: with one step each, batch 1 at context
// 4000 leaves 31 parts per unit to merge (32 query / 8 kv heads 14.9 -> 12.5 us, 64 / 8 at 4 bits 15.9 -> 12.7 us);
// with three the steps themselves get long (context 1000: 11.4 -> 11.9 us).
constexpr int kMinSteps = 2;

// resident: workgroups the device holds at once; stride, parts_limit: see the top; own_launch: the fp16 rows run in a
// launch of their own; one_row_part: which is not this kernel and leaves one part.  False: no cut fits.
inline bool cut_uniform(int64_t units, int tiles_a, int tiles_total, int resident, int stride, int parts_limit, bool own_launch,
                        bool one_row_part, UniformCut& cut) {
    const int n_a = (tiles_a + kStepTiles - 1) / kStepTiles, row_tiles = tiles_total - tiles_a;
    const int64_t total = units * n_a;
    const bool rows = row_tiles > 0;
    const int room = std::min(stride, parts_limit);
    if (total > 0x3fffffff || units > 0x1fffffff || (total == 0 && !rows)) return false;
    // Workgroups for a unit's fp16 rows: a wavefront per tile (a second tile is another 2-5 us in a chain that the
    // launch's end waits for) unless that takes more than a quarter of the residency, and at most half of the unit's
    // parts (a window of 8000 and more tokens asks for more than eight heads at 4 bits have).
    cut.row_split = std::max(1, std::min({(row_tiles + kStepTiles - 1) / kStepTiles, (int)std::max<int64_t>(1, resident / 4 / units), room / 2}));
    if (one_row_part) cut.row_split = 1;
    cut.row_wgs = rows ? (int)units * cut.row_split : 0;
    // One interval per workgroup that is resident beside the fp16 rows' (which end early), but not so short
    // that a unit would have more parts than there is room for.  With several workgroups per unit each
    // one's interval lies in one unit: a workgroup that straddles two enters and leaves both (4-7 us each, on the
    // critical path of the launch).  Otherwise all units are one axis (an interval of c steps cuts a unit into
    // at most (n_a - 1) / c + 2 parts).
    const int max_parts = room - (rows ? cut.row_split : 0);
    cut.unit_wgs = 0;
    cut.axis = StepAxis{1, 0};
    cut.intervals = 0;
    if (total == 0) return cut.row_split <= room;
    if (max_parts < 1) return false;
    int64_t n = std::min<int64_t>(own_launch ? resident : std::max(resident - cut.row_wgs, resident / 2), total);
    if (n >= 3 * units || max_parts == 1) {
        cut.unit_wgs = (int)std::min<int64_t>(max_parts, std::max<int64_t>(std::min<int64_t>(n / units, n_a / kMinSteps), 1));
        n = units * cut.unit_wgs;
        cut.axis = StepAxis{n_a / cut.unit_wgs, n_a % cut.unit_wgs};
    } else {
        while (n > 1 && std::min<int64_t>(n, (n_a - 1) / (total / n) + 2) > max_parts) n = std::min<int64_t>(n - 1, total / (total / n + 1));
        cut.axis = StepAxis{(int32_t)(total / n), (int32_t)(total % n)};
    }
    cut.intervals = n;
    return true;
}

// decode_one_kernel: workgroups per unit.  `steps`: of a unit; `room`: parts that fit (at least 1).  A part costs its unit
// about 4 us (workspace, counter, merge), so one workgroup per compute unit is enough unless each then has more than
// `many` steps: from there on the serial chain of its steps is the longer one, and two per compute unit -- or three, where two
// leave compute units with fewer workgroups than others -- are faster (2 bits, best number / one per compute unit: 32 units x
// 32 000 tokens 23 / 25 us, 64 x 32 000 39 / 42, 192 x 16 000 57 / 76, 320 x 8000 53 / 59; but 256 x 1000 11.2 against 13.1).
// A few more units than fit at once: halves, if they are long, so that the last ones do not run alone for as long (800 units x 4000
// tokens, 4 bits, 101 -> 96 us, 2 bits 70 -> 69; 2000 tokens 41.6 -> 45.8).  With more units beside them the last ones are alone for
// less long, and the line moves to longer units (896 units, whole / halves: 4 bits, 4127 tokens 118.0 / 113.3 us, 3000
// tokens 82.0 / 84.0; 2 bits 80.9 / 79.4 and 59.5 / 61.3), until whole units are the faster ones (960 units x 4000 tokens, 4 bits 107.1 / 111.1).
constexpr int kOneHeadMaxParts = 128;
inline int one_head_parts(int64_t units, int steps, int compute_units, int room, int many) {
    const int64_t cus = compute_units;
    int64_t w = std::max<int64_t>(1, cus / units);
    if (steps > many * w) {
        w = std::max<int64_t>(1, 2 * cus / units);
        if (units * w * 16 < 2 * cus * 15) w = std::max<int64_t>(1, 3 * cus / units);
        const bool halves = units * 8 <= 27 * cus ? steps > 2 * many : units * 2 <= 7 * cus && steps * 4 > 9 * many;
        if (units > 3 * cus && halves) w = 2;
    }
    return (int)std::max<int64_t>(1, std::min({w, (int64_t)steps, (int64_t)room}));
}

// Batches of different lengths: a sequence's units get as many workgroups as their steps ask for.  `total`: the steps of all units.  One
// workgroup per compute unit while none of them has more than `many` steps, as above; else one per two thirds of a compute unit's
// share of the steps, so that 256 units of one length are cut into halves and from 384 on such units are whole.  (Half of that share:
// 512 units of 3900-4100 tokens 52.3 us in place of 47.7, 4 bits 79.7 / 64.0, 320 of 2000 30.0 / 25.1..27.8; a third 56.0, 71.5, 29.0.  Three
// fifths and three quarters: 128 units of 500-16 000 tokens 30.8 and 33.9 us, 256 of 500-8000 35.8 and 31.5.)
inline int one_head_ragged_parts(int64_t total, int steps, int compute_units, int room, int many) {
    const int64_t cus = compute_units;
    const int64_t w = total <= many * cus ? (steps * cus + total - 1) / total : (3 * steps * cus + 2 * total - 1) / (2 * total);
    return (int)std::max<int64_t>(1, std::min({w, (int64_t)steps, (int64_t)room}));
}
// Such a batch of nearly one length (the shortest sequence has at least three quarters of the longest one's steps) and more than `many` steps
// per compute unit: every unit in as many parts as one_head_parts has for the longest, 0 where the rule above stays.  By the share a few
// of its numbers of units end just beyond whole workgroups per compute unit (182 units in three parts each: 546 on 256), or
// some sequences get a part more than others (384 units).  Share / this, 182 units: 12 600-14 000 tokens 56.7 / 48.7 us, 4 bits, 3600-4000 35.0 /
// 28.8; 100 x 11 700-13 000 32.0 / 29.4; 384 x 7200-8000 67.7 / 59.6.  It stays where this would end there in its turn, with three parts and more than two
// workgroups per compute unit: 200 units, 11 700-13 000 tokens, share 52.7, three parts 55.7; 220 x 7200-8000 38.4 / 40.7.
// A few more units than compute units, if long, in five parts, more than fit at once, where two or three parts end just beyond two or three workgroups
// per compute unit: two / five, 264 x 11 700-13 000 73.3 / 67.6 (4 bits 104.1 / 99.4), 280 x 8000 50.2 / 49.1; but 264 x 4000 31.3 / 32.3, 320 x 8000 51.6 / 53.0.
inline int one_head_near_parts(int64_t total, int64_t units, int longest, int shortest, int compute_units, int room, int many) {
    const int64_t cus = compute_units;
    if (total <= many * cus || (int64_t)shortest * 4 < (int64_t)longest * 3) return 0;
    if (units > cus && units * 6 <= 7 * cus && longest > 3 * many) return std::min({5, longest, room});
    const int parts = one_head_parts(units, longest, compute_units, room, many);
    return parts == 3 && units * parts > 2 * cus ? 0 : parts;
}
// What a workgroup of such a batch reads: its sequence's first workgroup (of all units, head by head), the sequence, workgroups per unit, counters
// after the step, steps of a unit.
struct OneHeadSequence { int32_t first_wg, sequence, parts, n_q, n_r, k_start, v_start, steps; };

// What decode_one_kernel's wavefronts take of a unit: the kernel's own arithmetic, here so that it can be walked without a device.
// A unit is n_kr tokens of fp16 rows, with UNEVEN the tokens from v_q (values in the cache) to n_kq, whose keys only are quantised, and
// `tiles` tiles.  An item is one wavefront's slot of a step: NT tokens' rows, MT tokens' key tile and value rows, or PT tiles.
// FLAT: items one after the other; otherwise rows are rounded to steps, then tiles.
template <int WV, int PT, int NT, int MT, int FLUSH_STEPS, bool FLUSH, bool UNEVEN>
struct OneHeadWork {
    static constexpr bool FLAT = FLUSH || UNEVEN;
    static constexpr int kTiles = WV * PT, kRows = WV * NT;        // of a step
    int s0, m0, a0, len_a, all_rows, all_fp16, turn, rot, lead;
    int n_row_items, n_fp16_items, n_items;                        // of this part: rows; and those of MT tokens; and tiles

    // steps of a unit; with FLUSH the last FLUSH_STEPS are the flush, which no item stands for
    static KIVI_HOST_DEVICE int steps(int tiles, int n_kq, int v_q, int n_kr) {
        if (!FLAT) return (tiles + kTiles - 1) / kTiles + (n_kr + kRows - 1) / kRows;
        const int fp16 = (n_kr + NT - 1) / NT + (UNEVEN ? (n_kq - (v_q & -MT)) / MT : 0);
        return (fp16 + (tiles + PT - 1) / PT + WV - 1) / WV + (FLUSH ? FLUSH_STEPS : 0);
    }
    // part `part` of `parts`; order() completes it (apart, so that the kernel computes that where it needs it: in one, steps that flush
    // took 0.8 % more)
    KIVI_HOST_DEVICE OneHeadWork(StepAxis axis, int part, int parts, int tiles, int n_kq, int v_q, int n_kr) {
        const int real = axis.start(parts) - (FLUSH ? FLUSH_STEPS : 0), s1 = least(axis.start(part + 1), real);
        s0 = least(axis.start(part), real);
        const int nr = (n_kr + kRows - 1) / kRows;
        a0 = most(s0 - nr, 0);
        len_a = most(s1 - nr, 0) - a0;
        m0 = v_q & -MT;
        all_rows = (n_kr + NT - 1) / NT;
        all_fp16 = all_rows + (UNEVEN ? (n_kq - m0) / MT : 0);
        n_items = FLAT ? most(least(s1 * WV, all_fp16 + (tiles + PT - 1) / PT) - s0 * WV, 0) : (s1 - s0) * WV;
        n_row_items = FLAT ? least(most(all_rows - s0 * WV, 0), n_items) : least(most(nr - s0, 0), s1 - s0) * WV;
        n_fp16_items = UNEVEN ? least(most(all_fp16 - s0 * WV, 0), n_items) : n_row_items;
    }
    // u: the unit; flush_lead: items that each other wavefront takes before the one that flushes (the last one of the last part)
    // takes its first
    KIVI_HOST_DEVICE void order(int part, int parts, int u, int flush_lead) {
        // Tiles in an order rotated by the unit: workgroups in lockstep that all read the same relative offset of their units
        // would meet on few memory channels for unlucky strides (a copy alone: 32.3 -> 29.8 us at 512 units).
        turn = FLAT ? n_items - n_fp16_items : len_a;
        rot = turn > 0 ? (int)((uint32_t)(u * (FLUSH ? WV : 5)) % (uint32_t)turn) : 0;
        lead = FLUSH && part == parts - 1 ? (WV - 1) * flush_lead : 0;
    }
    // A wavefront takes every WV-th item; in the workgroup that flushes, whose last wavefront comes late, the others have the first
    // `lead` items to themselves.  (The shares are fixed: sums in the same order every time.)
    KIVI_HOST_DEVICE int first(int wave, bool flushes) const { return flushes ? lead + wave : wave; }
    KIVI_HOST_DEVICE int after(int item) const { return item + (item < lead ? WV - 1 : WV); }
    // an item's first token of the window, token, and tile
    KIVI_HOST_DEVICE int row_of(int item) const { return (s0 + item / WV) * kRows + item % WV * NT; }
    KIVI_HOST_DEVICE int mixed_of(int item) const { return m0 + (s0 * WV + item - all_rows) * MT; }
    KIVI_HOST_DEVICE int tile_of(int item) const {
        if (FLAT) {
            int a = item - n_fp16_items + rot;
            a -= a >= turn ? turn : 0;
            return (s0 * WV + n_fp16_items - all_fp16 + a) * PT;
        }
        int a = (item - n_row_items) / WV + rot;
        a -= a >= len_a ? len_a : 0;
        return (a0 + a) * kTiles + item % WV * PT;
    }

private:
    static KIVI_HOST_DEVICE int least(int a, int b) { return a < b ? a : b; }
    static KIVI_HOST_DEVICE int most(int a, int b) { return a > b ? a : b; }
};

// the two bit widths' slots (decode_one_kernel checks that they are its own)
template <int BITS, bool FLUSH, bool UNEVEN>
using OneHeadItems = OneHeadWork<4, BITS == 2 ? 2 : 1, BITS == 2 ? 12 : 10, BITS == 2 ? 16 : 8, BITS == 2 ? 1 : 2, FLUSH, UNEVEN>;

}  // namespace kivi
