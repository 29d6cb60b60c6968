"""bf16 calls over short lists (one work group per (cell, KV head)) against the
fp64 oracle, at the edges of tiles and of the route, and against the
shared-prompt kernel that an explicit split takes; forked sweeps included
(their dormant cells are checked in test_gpu_forked.py, whose tiny cases take
this route too)."""
import numpy as np
import pytest
import torch

import gpu_common as gc
import paper_2605_30574_amd as sp
import workloads
from test_gpu_forked import check_forked
from workloads import DONOR_BLANK, DONOR_DIFF, DONOR_ZERO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sp.load_library()


def _w(C, Hq, Hkv, D, Tp, span, donor, window=0, steps=300):
    N = 4
    cells = tuple((i % (N + 1), (0, 2, 9)[i % 3]) for i in range(C))
    return workloads.get("qwen3-4b").with_(n_layers=N, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, prompt_len=Tp, span=span,
                                           n_steps=steps, cells=cells, donor=donor, scale=D ** -0.5,
                                           local_window=window)


# list lengths around the limits (384, 160, 64 keys at D = 128 for one, two and
# three work groups a compute unit, 224 and 96 at D = 256), spans off tile edges
CASES = [
    (_w(3, 8, 2, 128, 17, (3, 14), DONOR_BLANK), (0, 14, 15, 299)),
    (_w(5, 32, 8, 128, 256, (40, 236), DONOR_DIFF), (0, 127, 128)),
    (_w(9, 2, 2, 64, 100, (0, 100), DONOR_ZERO), (1, 31, 283, 284)),
    (_w(7, 16, 2, 64, 33, (1, 32), DONOR_BLANK, window=20), (0, 5, 40)),
    (_w(6, 8, 4, 256, 40, (7, 33), DONOR_BLANK), (3, 183, 184)),
    (_w(65, 8, 8, 128, 48, (5, 45), DONOR_ZERO, steps=120), (4, 111, 112)),
    (_w(80, 32, 8, 64, 31, (2, 30), DONOR_DIFF, steps=80), (0, 32, 33)),
    (_w(4, 8, 1, 256, 0, (0, 0), DONOR_BLANK), (0, 222)),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_short_lists(i):
    w, steps = CASES[i]
    lw = workloads.cell_lw(w)
    layer = 2
    bufs = gc.gpu_layer(w, layer)
    hb = gc.host(bufs)
    for step in steps:
        q = workloads.make_q(w, layer, step, device="cuda")
        gc.announce(f"direct case {i} step={step}")
        out, lse = gc.run_attn(w, layer, step, bufs, q, lw)
        ref_o, ref_l = gc.run_oracle(w, layer, step, hb, workloads.to_numpy(q), lw)
        gc.assert_attn_close(out, lse, ref_o, ref_l, f"case {i} step {step}")
        o2, l2 = gc.run_attn(w, layer, step, bufs, q, lw)
        assert np.array_equal(out, o2) and np.array_equal(lse, l2), "repeat call"
        o3, l3 = gc.run_attn(w, layer, step, bufs, q, lw, split=64)
        gc.assert_attn_close(o3, l3, out, lse, f"case {i} step {step}: split")
        if w.donor != DONOR_ZERO and w.prompt_len:   # a splice moves no tile boundary
            never = np.array([[w.n_layers, 0]] * w.n_cells, dtype=np.int32)
            same = dict(bufs, donor_k=bufs["clean_k"], donor_v=bufs["clean_v"])
            o_u, l_u = gc.run_attn(w, layer, step, bufs, q, never)
            o_s, l_s = gc.run_attn(w, layer, step, same, q, lw)
            assert np.array_equal(o_u, o_s) and np.array_equal(l_u, l_s)


@pytest.mark.parametrize("D,Hkv", [(64, 2), (128, 8), (256, 4)])
def test_forked_short_lists(D, Hkv):
    w = _w(11, 4 * Hkv, Hkv, D, 50, (4, 47), DONOR_BLANK, steps=60)
    lw = np.ascontiguousarray(np.concatenate([workloads.cell_lw(w), [[w.n_layers, 0]]]).astype(np.int32))
    for step in (0, 1, 2, 8, 9, 30):
        check_forked(w, 1, step, lw, lw.shape[0] - 1, f"direct forked D={D}")


def test_the_workspace_is_still_asked_for():
    w = CASES[1][0]
    lw = workloads.cell_lw(w)
    bufs = gc.gpu_layer(w, 2)
    shape, call = gc.shape_of(w), sp.make_call(2, 0, 0, w.scale)
    need = sp.splice_decode_attn_workspace_bytes(shape, call)
    ws = torch.empty(need // 2 // 256 * 256, dtype=torch.uint8, device="cuda")
    sp.splice_workspace_init(ws)
    with pytest.raises(sp.SpliceError) as e:
        gc.run_attn(w, 2, 0, bufs, workloads.make_q(w, 2, 0, device="cuda"), lw, ws=ws)
    assert e.value.status == sp.SPLICE_EWORKSPACE
