"""The host-side plan (csrc/plan.hpp), compiled here for the CPU: where calls
keep their counters and partial results, and which route they take."""
import ctypes
import itertools
import os
import subprocess

import pytest

import paper_2605_30574_amd as sp
from paper_2605_30574_amd import splice as S

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "plan.hpp"
using namespace splice;
extern "C" {
// counters [0, 1), partial results [2, 3), the array's size [4] of a call that fits the no-allocation entry's limit; 0 if none
int noalloc_ranges(const splice_shape *sh, const splice_call *call, int64_t *r) {
    if (validate_shape(sh) != SPLICE_OK || validate_call(*sh, call) != SPLICE_OK) return 0;
    const Geometry geo = geometry(*sh, *call);
    const AttnPlan p = plan_from_geo(*sh, *call, geo, sh->n_cells / 2, sh->n_cells);
    if (p.n_slots < 1 || workspace_layout(*sh, p.n_slots).total > SPLICE_NOALLOC_WORKSPACE_BYTES) return 0;
    const WorkspaceLayout w = noalloc_layout(*sh, p.n_slots);
    r[0] = w.counters_off; r[1] = r[0] + (int64_t)sh->n_cells * sh->n_kv_heads * 4;
    r[2] = w.part_off; r[3] = r[2] + w.part_bytes; r[4] = kNoallocBytes;
    return 1;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2605_30574_amd", "csrc"), "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so))


def _shape(C, Hkv, G, D, Tp, dtype="bf16", cap=64):
    return sp.make_shape(C, 4, Hkv * G, Hkv, D, Tp, (0, Tp // 2), cap, False, dtype)


def test_no_call_leaves_partials_where_another_keeps_counters(plan):
    """The no-allocation entry's array is shared by calls of every shape."""
    ranges = []
    for C, Hkv, G, D, Tp, dt in itertools.product((1, 8, 9, 64, 255, 256), (1, 8, 32, 200), (1, 8), (64, 256),
                                                  (0, 400, 8192), ("bf16", "f32")):
        r = (ctypes.c_int64 * 5)()
        for split in (0, 64):
            if plan.noalloc_ranges(ctypes.byref(_shape(C, Hkv, G, D, Tp, dt)), ctypes.byref(
                    sp.make_call(0, 5, 0, 1.0, split)), r):
                ranges.append(tuple(r))
    assert len(ranges) > 150
    last_counter, first_part = max(r[1] for r in ranges), min(r[2] for r in ranges)
    assert last_counter <= first_part, (last_counter, first_part)
    assert all(S.SPLICE_NOALLOC_WORKSPACE_BYTES < r[4] and r[3] <= r[4] for r in ranges)
