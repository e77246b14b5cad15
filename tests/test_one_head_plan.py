"""How decode_one_kernel's work is cut (csrc/kivi_tiles_plan.h), compiled for the host: one_head_parts, and OneHeadWork, whose arithmetic
is the kernel's own, walked as its wavefronts walk it.  Whatever the lengths, every row of the window, every token with a quantised
key and an fp16 value, and every tile is taken exactly once, and no part is empty of steps or past the workspace's rows."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "kivi_tiles_plan.h"
using namespace kivi;
namespace {
constexpr int WV = 4;
std::vector<int> rows, mixed, tile;
// 0, or what is wrong.  v_q: tokens with quantised values, a multiple of 32 unless UNEVEN; n_kq >= v_q
template <int BITS, bool FLUSH, bool UNEVEN>
int check(int64_t units, int u, int n_kq, int v_q, int n_kr, int cus, int room, int flush_lead) {
    using Work = OneHeadItems<BITS, FLUSH, UNEVEN>;
    constexpr int PT = Work::kTiles / WV, NT = Work::kRows / WV, MT = BITS == 2 ? 16 : 8, many = BITS == 2 ? 8 : 12;
    const int tiles = (v_q + 31) / 32, steps = Work::steps(tiles, n_kq, v_q, n_kr);
    if (steps < 1) return 0;
    const int parts = one_head_parts(units, steps, cus, room, many);
    if (parts < 1 || parts > room || parts > steps) return 1;
    const StepAxis axis{steps / parts, steps % parts};
    if (axis.start(parts) != steps) return 2;
    rows.assign(n_kr, 0);
    mixed.assign(n_kq, 0);
    tile.assign(tiles, 0);
    for (int part = 0; part < parts; ++part) {
        if (axis.start(part + 1) <= axis.start(part)) return 3;
        Work w(axis, part, parts, tiles, n_kq, v_q, n_kr);
        w.order(part, parts, u, flush_lead);
        if (w.n_row_items < 0 || w.n_row_items > w.n_fp16_items || w.n_fp16_items > w.n_items) return 4;
        if (!FLUSH && w.n_items < 1) return 5;
        std::vector<int> taken(w.n_items, 0);
        for (int wave = 0; wave < WV; ++wave)
            for (int item = w.first(wave, FLUSH && part == parts - 1 && wave == WV - 1); item < w.n_items; item = w.after(item)) {
                if (taken[item]++) return 6;
                if (item < w.n_row_items) {                      // rows; past the window's end nothing
                    for (int t = w.row_of(item); t < std::min(w.row_of(item) + NT, n_kr); ++t)
                        if (t < 0 || rows[t]++) return 7;
                } else if (item < w.n_fp16_items) {
                    const int t0 = w.mixed_of(item);             // of one key tile, which is there
                    if (t0 < 0 || t0 % MT || t0 + MT > n_kq || t0 / 32 != (t0 + MT - 1) / 32) return 8;
                    for (int t = std::max(t0, v_q); t < t0 + MT; ++t)
                        if (mixed[t]++) return 9;
                } else {
                    for (int t = w.tile_of(item); t < std::min(w.tile_of(item) + PT, tiles); ++t)
                        if (t < 0 || tile[t]++) return 10;
                }
            }
        for (int n : taken)
            if (n != 1) return 11;
    }
    for (int n : rows)
        if (n != 1) return 12;
    for (int t = 0; t < n_kq; ++t)
        if (mixed[t] != (UNEVEN && t >= v_q)) return 13;
    for (int n : tile)
        if (n != 1) return 14;
    return 0;
}
template <int BITS>
int check_form(int form, int64_t units, int u, int n_kq, int v_q, int n_kr, int cus, int room, int flush_lead) {
    return form == 0   ? check<BITS, false, false>(units, u, n_kq, v_q, n_kr, cus, room, flush_lead)
           : form == 1 ? check<BITS, true, false>(units, u, n_kq, v_q, n_kr, cus, room, flush_lead)
                       : check<BITS, false, true>(units, u, n_kq, v_q, n_kr, cus, room, flush_lead);
}
}
// batches of different lengths: steps -> workgroups per unit; 0, or what is wrong
extern "C" int check_ragged(const int* steps, int sequences, int heads, int cus, int room, int many) {
    int64_t total = 0, wgs = 0, longest = 0;
    for (int b = 0; b < sequences; ++b) total += (int64_t)steps[b] * heads;
    for (int b = 0; b < sequences; ++b) {
        const int parts = one_head_ragged_parts(total, steps[b], cus, room, many);
        if (parts < 1 || parts > room || parts > steps[b]) return 1;
        const StepAxis axis{steps[b] / parts, steps[b] % parts};
        if (axis.len < 1 || axis.start(parts) != steps[b]) return 2;
        if (parts < room) longest = std::max<int64_t>(longest, axis.len + (axis.rem > 0));
        wgs += (int64_t)parts * heads;
    }
    if (longest * (total <= (int64_t)many * cus ? cus : 3 * cus / 2) > total + longest * 3 * cus / 2) return 3;      // longer than its share, rounded up
    if (wgs > (int64_t)sequences * heads + 2 * (int64_t)cus) return 4;
    return 0;
}
extern "C" int near_parts(int64_t total, int64_t units, int longest, int shortest, int cus, int room, int many) {
    return one_head_near_parts(total, units, longest, shortest, cus, room, many);
}
// form 0: K and V split alike, 1: with a flush, 2: split differently
extern "C" int check_all(int bits, int form, int n_kq, int v_q, int n_kr, int* at) {
    const int units[] = {1, 2, 3, 8, 31, 32, 85, 86, 128, 255, 256, 257, 320, 512, 767, 768, 769, 800, 864, 865, 896, 897, 2048};
    int turn = 0;
    for (int count : units)
        for (int room : {1, 3, 128})
            for (int cus : {256, 7}) {
                const int u = turn++ % count, lead = turn % 7;
                const int e = bits == 2 ? check_form<2>(form, count, u, n_kq, v_q, n_kr, cus, room, lead)
                                        : check_form<4>(form, count, u, n_kq, v_q, n_kr, cus, room, lead);
                if (e) { at[0] = count; at[1] = room; at[2] = cus; return e; }
            }
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("one_head_plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-include", "algorithm", "-include", "vector", "-include", "cstdint",
                    "-I", os.path.join(ROOT, "paper_2402_02750_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan.so")], check=True)
    return ctypes.CDLL(str(d / "plan.so"))


@pytest.mark.parametrize("heads", [1, 4, 40])
@pytest.mark.parametrize("steps", [[1], [300], [1, 1, 300], [16] * 64, list(range(1, 193)), [5000, 1, 2, 3], [7] * 4000])
def test_ragged_parts(plan, steps, heads):
    arr = (ctypes.c_int * len(steps))(*steps)
    for cus in (256, 7):
        for room in (1, 2, 128):
            for many in (8, 12):
                assert plan.check_ragged(arr, len(steps), heads, cus, room, many) == 0, f"{cus} compute units, {room} rows, {many}"


@pytest.mark.parametrize("cus", [256, 7])
def test_near_parts(plan, cus):
    """Batches of nearly one length and many steps: as many parts as fit and there are steps; other batches keep the share."""
    plan.near_parts.argtypes = [ctypes.c_int64] * 2 + [ctypes.c_int] * 5
    for units in range(1, 5 * cus, max(1, cus // 40)):
        for longest in (1, 9, 20, 31, 53, 300):
            for room in (1, 2, 128):
                total = units * longest
                parts = plan.near_parts(total, units, longest, longest - longest // 4, cus, room, 8)
                assert 0 <= parts <= min(room, longest) and (parts == 0 or total > 8 * cus)
                assert parts == 0 or units * parts <= max(3 * cus, 2 * units, 35 * cus // 6 if longest > 24 else 0)
                assert plan.near_parts(total, units, longest, (longest * 3 - 1) // 4, cus, room, 8) == 0
    assert [plan.near_parts(u * 53, u, 53, 48, 256, 128, 8) for u in (171, 182, 192, 193, 239, 240, 256, 257, 298, 299, 384)] == [4, 4, 4, 0, 0, 2, 2, 5, 5, 2, 2]
    assert plan.near_parts(264 * 24, 264, 24, 20, 256, 128, 8) == 2


TILES = list(range(0, 12)) + [15, 16, 17, 31, 63, 64, 65, 128, 1000]


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("form", ["alike", "flush", "uneven"])
def test_every_item_once(plan, bits, form):
    at = (ctypes.c_int * 3)()
    for tiles in TILES:
        for window in [*range(form == "flush", 64 if tiles < 3 else 1), *range(1, 200, 11), 479, 1024]:
            if form == "uneven":
                # from no value row more than the window's to a window's worth; any position in a tile
                cases = [(32 * tiles, v, window) for v in {max(0, 32 * tiles - d) for d in (0, 1, 7, 8, 31, 32, 33, 127, 128, 4000)}]
            else:
                cases = [(32 * tiles, 32 * tiles, window)]
            for n_kq, v_q, n_kr in cases:
                error = plan.check_all(bits, ["alike", "flush", "uneven"].index(form), n_kq, v_q, n_kr, at)
                assert error == 0, f"error {error}: {n_kq} keys, {v_q} values, {n_kr} rows; units, rows, compute units {list(at)}"
