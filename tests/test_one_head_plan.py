"""How decode_one_kernel's work is cut (csrc/kivi_tiles_plan.h), compiled for the host: whatever the lengths, every item -- rows,
key tiles with value rows, tiles -- lies in exactly one part, and no part is empty of steps or past the workspace's rows."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "kivi_tiles_plan.h"
using namespace kivi;
// as the kernel: `items` in steps of four, the last `flush` steps not handed out; 0, or what is wrong
static int check(int64_t units, int items, int flush, int cus, int room, int many) {
    const int steps = (items + 3) / 4 + flush;
    if (steps < 1) return 0;
    const int w = one_head_parts(units, steps, cus, room, many);
    if (w < 1 || w > room || w > steps) return 1;
    const StepAxis axis{steps / w, steps % w};
    const int real = axis.start(w) - flush;
    if (axis.start(w) != steps) return 2;
    int done = 0;
    for (int part = 0; part < w; ++part) {
        const int s0 = std::min(axis.start(part), real), s1 = std::min(axis.start(part + 1), real);
        if (axis.start(part + 1) <= axis.start(part)) return 3;
        const int n = s0 == s1 ? 0 : std::min(s1 * 4, items) - s0 * 4;      // (a part may hold nothing but the flush)
        if (n < 0 || (n == 0 && !flush)) return 4;
        if (n > 0 && s0 * 4 != done) return 5;
        done += n;
    }
    return done == items ? 0 : 6;
}
extern "C" int check_all(int items_max, int flush, int many, int* at) {
    const int units[] = {1, 2, 3, 8, 31, 32, 85, 86, 128, 255, 256, 257, 320, 512, 767, 768, 769, 800, 864, 865, 896, 897, 2048};
    const int rooms[] = {1, 2, 3, 8, 31, 128};
    for (int items = flush ? 0 : 1; items <= items_max; ++items)
        for (int u : units)
            for (int room : rooms)
                for (int cus : {256, 304, 7})
                    if (const int e = check(u, items, flush, cus, room, many)) { at[0] = items; at[1] = u; at[2] = room; return e; }
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("one_head_plan")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-include", "algorithm", "-include", "vector", "-include", "cstdint",
                    "-I", os.path.join(ROOT, "paper_2402_02750_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan.so")], check=True)
    return ctypes.CDLL(str(d / "plan.so"))


@pytest.mark.parametrize("flush,many", [(0, 8), (0, 12), (1, 8), (2, 12)])
def test_every_item_once(plan, flush, many):
    at = (ctypes.c_int * 3)()
    error = plan.check_all(1500, flush, many, at)
    assert error == 0, f"error {error}: items, units, rows {list(at)}"
