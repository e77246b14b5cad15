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

// An axis of steps in intervals of `len`, the first `rem` of them one step longer.
struct StepAxis {
    int32_t len, rem;
    KIVI_HOST_DEVICE int start(int g) const { return g * len + (g < rem ? g : rem); }
    KIVI_HOST_DEVICE int owner(int pos) const {
        const int cut = rem * (len + 1);
        return pos < cut ? (int)((uint32_t)pos / (uint32_t)(len + 1)) : rem + (int)((uint32_t)(pos - cut) / (uint32_t)len);
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
    bool whole_units = false;          // room for a single part: every workgroup takes whole units
    // {first unit, first step in it, steps, 0} per workgroup, then the steps before each sequence
    static constexpr int kWords = 4;
};

// steps[b]: steps of each of the n_kv_heads units of sequence b (at least 1); rows: parts per head that fit, row 0
// included (at least 2).  Appends the table to `out`.
inline RaggedCut cut_ragged(const std::vector<int32_t>& steps, int n_kv_heads, int64_t max_workgroups, int rows, std::vector<int32_t>& out) {
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
    cut.axis = StepAxis{(int32_t)(total / cut.workgroups), (int32_t)(total % cut.workgroups)};

    const size_t base = out.size();
    out.resize(base + (size_t)cut.workgroups * RaggedCut::kWords + steps.size(), 0);
    int32_t* desc = out.data() + base;
    int32_t* before = desc + (size_t)cut.workgroups * RaggedCut::kWords;
    int64_t cum = 0, g = 0;
    for (size_t b = 0; b < steps.size(); ++b) {
        const int64_t n = steps[b], unit0 = (int64_t)b * n_kv_heads, end = cum + n * n_kv_heads;
        before[b] = (int32_t)cum;
        for (; g < cut.workgroups; ++g) {
            int64_t begin = cut.axis.start((int)g), length = cut.axis.start((int)g + 1) - begin;
            if (cut.whole_units) {
                const int64_t u0 = g * units / cut.workgroups, u1 = (g + 1) * units / cut.workgroups;
                if (u0 >= unit0 + n_kv_heads) break;
                begin = cum + (u0 - unit0) * n;
                length = 0;
                for (int64_t u = u0; u < u1; ++u) length += steps[(size_t)(u / n_kv_heads)];
            }
            if (begin >= end) break;
            desc[4 * g + 0] = (int32_t)(unit0 + (begin - cum) / n);
            desc[4 * g + 1] = (int32_t)((begin - cum) % n);
            desc[4 * g + 2] = (int32_t)length;
        }
        cum = end;
    }
    return cut;
}

}  // namespace kivi
