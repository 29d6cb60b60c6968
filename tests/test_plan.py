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
    if (p.n_slots < 1 || p.bytes > SPLICE_NOALLOC_WORKSPACE_BYTES) return 0;
    const WorkspaceLayout w = noalloc_layout(*sh, p.n_slots);
    r[0] = w.counters_off; r[1] = r[0] + (int64_t)sh->n_cells * sh->n_kv_heads * 4;
    r[2] = w.part_off; r[3] = r[2] + w.part_bytes; r[4] = kNoallocBytes;
    return 1;
}
// f32: 1 where the call takes the shared-prompt route
int takes_wide(const splice_shape *sh, const splice_call *call) {
    return plan_from_geo(*sh, *call, geometry(*sh, *call), sh->n_cells / 2, sh->n_cells).wide;
}
// workspace bytes of the call's plan [0] and of the plan without that route [1], chunks [2] and their length [3], where
// its partial results lie [4, 5)
void plan_bytes(const splice_shape *sh, const splice_call *call, int64_t *r) {
    const Geometry geo = geometry(*sh, *call);
    const AttnPlan p = plan_from_geo(*sh, *call, geo, 0, sh->n_cells);
    const AttnPlan q = plan_from_geo(*sh, *call, geo, 0, sh->n_cells, Residency(), true, false);
    r[0] = p.bytes; r[1] = q.bytes; r[2] = p.n_p; r[3] = p.p_len;
    const WorkspaceLayout w = workspace_layout(*sh, p.n_slots, p.wide);
    r[4] = w.part_off; r[5] = w.total;
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


# (cells, KV heads, G, D, prompt keys): measured on both routes, see wide_f32 in plan.hpp
@pytest.mark.parametrize("dims,wide", [
    ((8, 1, 4, 128, 8349), False), ((29, 1, 4, 128, 1638), False), ((9, 1, 4, 64, 3964), False),
    ((9, 4, 4, 256, 1528), False), ((49, 1, 4, 256, 3146), False), ((9, 1, 8, 128, 2988), False),
    ((27, 8, 4, 64, 422), False), ((50, 4, 4, 128, 435), False), ((51, 4, 4, 256, 417), False),
    ((69, 4, 4, 128, 446), True), ((67, 4, 4, 64, 450), True), ((84, 1, 4, 128, 4544), True), ((25, 4, 4, 64, 2917), True), ((39, 4, 4, 256, 651), True),
    ((17, 2, 4, 64, 1239), False), ((29, 1, 8, 64, 5749), True), ((6, 1, 8, 128, 605), True), ((79, 4, 1, 128, 1813), True),
    ((59, 1, 8, 128, 3821), True), ((64, 8, 4, 128, 1024), True), ((46, 8, 1, 128, 4360), True)])
def test_f32_route_needs_rows_for_the_whole_gpu(plan, dims, wide):
    assert plan.takes_wide(ctypes.byref(_shape(*dims, dtype="f32")), ctypes.byref(sp.make_call(0, 5, 0, 1.0))) == wide


def test_both_entries_take_one_f32_plan(plan):
    """The shared-prompt route never asks for more than the no-allocation array
    holds, nor for other bytes than the query says, so no call's route (and so
    no call's bits) depends on its workspace, and what that entry accepts is
    what it accepted without the route."""
    wide, limit = 0, S.SPLICE_NOALLOC_WORKSPACE_BYTES
    call = sp.make_call(0, 5, 0, 1.0)
    for C, Hkv, G, D, Tp in itertools.product((5, 8, 64, 128, 256), (1, 8, 24), (1, 2, 4, 8), (64, 128, 256),
                                              (400, 1000, 4096, 32768)):
        sh = _shape(C, Hkv, G, D, Tp, "f32")
        r = (ctypes.c_int64 * 6)()
        plan.plan_bytes(ctypes.byref(sh), ctypes.byref(call), r)
        assert r[0] == sp.splice_decode_attn_workspace_bytes(sh, call) <= sp.splice_decode_attn_workspace_bytes(sh)
        assert (r[0] <= limit) == (r[1] <= limit), (C, Hkv, G, D, Tp, list(r))
        if plan.takes_wide(ctypes.byref(sh), ctypes.byref(call)):
            wide += 1
            assert r[0] >= max(r[1], r[5]) and r[4] >= 256 + 4 * 256 * Hkv   # behind any cell count's counters
            assert 1 <= r[2] <= 16 and r[2] * r[3] >= Tp > (r[2] - 1) * r[3] and r[3] % 32 == 0
    assert wide > 200, wide
