"""float32 calls over a shared prompt on the fp32 matrix cores, against the
fp64 oracle and against the general route.

The products and sums are fp32, as on the general route: both are off by 2e-7
to 3e-7 of the outputs in the 2-norm, and single outputs by 1.1e-6 of the largest
at most, as measured at every size here; 6e-6 leaves a factor of five, and is a
hundredth of what weights or products of 11 bits would give."""
import numpy as np
import pytest
import torch

import gpu_common as gc
import paper_2605_30574_amd as sp
import workloads
from workloads import DONOR_BLANK, DONOR_DIFF, DONOR_ZERO

pytestmark = pytest.mark.gpu
REL = 6e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sp.load_library()


def _close(out, ref):
    return np.abs(out - ref).max() <= REL * np.abs(ref).max()


def _w(C, Hq, Hkv, D, Tp, span, donor, window=0, steps=20):
    N = 4
    cells = tuple((i % (N + 1), (0, 2, 9)[i % 3]) for i in range(C))
    return workloads.get("qwen3-4b").with_(n_layers=N, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, prompt_len=Tp, span=span,
                                           n_steps=steps, cells=cells, donor=donor, dtype="f32", scale=D ** -0.5,
                                           local_window=window)


# rows that fill and do not fill a 64-row group, prompts that end inside a tile
# and a chunk, spans on and off tile edges, every donor, a window, every head size
CASES = {
    "d128-g4": (8, 32, 8, 128, 512, (40, 480), DONOR_BLANK),
    "d128-g4-ragged": (17, 8, 2, 128, 1031, (33, 999), DONOR_DIFF),
    "d128-g4-zero": (9, 8, 2, 128, 777, (16, 776), DONOR_ZERO),
    "d128-g4-window": (16, 8, 2, 128, 900, (100, 800), DONOR_BLANK, 500),
    "d64-g8": (5, 16, 2, 64, 530, (3, 529), DONOR_BLANK),
    "d64-g8-zero-full": (33, 8, 1, 64, 1300, (0, 1300), DONOR_ZERO),
    "d256-g2": (33, 16, 8, 256, 769, (64, 700), DONOR_DIFF),
    "d256-g4": (8, 4, 1, 256, 400, (7, 391), DONOR_BLANK),
    "d64-g1": (64, 4, 4, 64, 1537, (1, 1536), DONOR_BLANK),
    # the same edges with rows enough for the route (192 over all KV heads at D = 64, else 320)
    "d128-g4-ragged-rows": (41, 8, 2, 128, 1031, (33, 999), DONOR_DIFF),
    "d128-g4-zero-rows": (80, 8, 2, 128, 777, (16, 776), DONOR_ZERO),
    "d128-g4-window-rows": (47, 8, 2, 128, 900, (100, 800), DONOR_BLANK, 500),
    "d64-g8-rows": (25, 16, 2, 64, 530, (3, 529), DONOR_BLANK),
    "d256-g4-rows": (81, 4, 1, 256, 400, (7, 391), DONOR_BLANK),
    "d64-g1-rows": (80, 4, 4, 64, 1537, (1, 1536), DONOR_BLANK),
}


@pytest.mark.parametrize("name", CASES)
def test_shared_prompt_route(name):
    w = _w(*CASES[name])
    lw = workloads.cell_lw(w)
    shape = gc.shape_of(w)
    for layer, step in ((0, 0), (2, 5), (3, 19)):
        bufs = gc.gpu_layer(w, layer)
        hb = gc.host(bufs)
        q = workloads.make_q(w, layer, step, device="cuda")
        call = sp.make_call(layer, step, w.window(layer), w.scale)
        gc.announce(f"wide f32 {name} layer={layer} step={step}")
        out, lse = gc.run_attn(w, layer, step, bufs, q, lw)
        ref_o, ref_l = gc.run_oracle(w, layer, step, hb, workloads.to_numpy(q), lw)
        assert _close(out, ref_o) and np.abs(lse - ref_l).max() <= 1e-5 * max(1.0, np.abs(ref_l).max())
        o2, l2 = gc.run_attn(w, layer, step, bufs, q, lw)
        assert np.array_equal(out, o2) and np.array_equal(lse, l2), "repeat call"
        # a workspace of just the bytes asked for gives the same bits, a smaller one is refused
        need = sp.splice_decode_attn_workspace_bytes(shape, call)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        sp.splice_workspace_init(ws)
        o3, l3 = gc.run_attn(w, layer, step, bufs, q, lw, ws=ws)
        assert np.array_equal(out, o3) and np.array_equal(lse, l3)
        with pytest.raises(sp.SpliceError) as e:
            gc.run_attn(w, layer, step, bufs, q, lw, ws=ws[: need - 256])
        assert e.value.status == sp.SPLICE_EWORKSPACE
        o4, _ = gc.run_attn(w, layer, step, bufs, q, lw, split=256)
        assert _close(o4, ref_o)


@pytest.mark.parametrize("C", [16, 40])   # the general route, the shared-prompt one
def test_donor_equal_clean_is_unspliced_up_to_grouping(C):
    """Spliced and unspliced cells sit in different row groups, which share no
    arithmetic: the bits of a cell depend on neither."""
    w = _w(C, 8, 2, 128, 700, (40, 650), DONOR_BLANK)
    lw = workloads.cell_lw(w)
    never = np.array([[w.n_layers, 0]] * w.n_cells, dtype=np.int32)
    bufs = gc.gpu_layer(w, 2)
    same = dict(bufs, donor_k=bufs["clean_k"], donor_v=bufs["clean_v"])
    q = workloads.make_q(w, 2, 5, device="cuda")
    gc.announce("wide f32 donor == clean")
    o_u, l_u = gc.run_attn(w, 2, 5, bufs, q, never)
    o_s, l_s = gc.run_attn(w, 2, 5, same, q, lw)
    # a spliced cell's list is cut at the span's edges, an unspliced cell's too
    assert np.array_equal(o_u, o_s) and np.array_equal(l_u, l_s)


def test_many_short_lists():
    """Cellwise calls with two work groups a compute unit and fewer."""
    for C, Hkv, G in ((128, 4, 4), (64, 8, 4), (40, 2, 4), (6, 1, 8)):
        w = _w(C, Hkv * G, Hkv, 64, 37, (3, 30), DONOR_BLANK)
        lw = workloads.cell_lw(w)
        bufs = gc.gpu_layer(w, 1)
        q = workloads.make_q(w, 1, 19, device="cuda")
        gc.announce(f"cellwise C={C} Hkv={Hkv} G={G}")
        out, lse = gc.run_attn(w, 1, 19, bufs, q, lw)
        ref_o, ref_l = gc.run_oracle(w, 1, 19, gc.host(bufs), workloads.to_numpy(q), lw)
        assert _close(out, ref_o) and np.abs(lse - ref_l).max() <= 1e-5 * max(1.0, np.abs(ref_l).max())


# long and short chunks (the first: 1250 keys each), a full merge of 17 slots,
# every head size and few and many rows a KV head
@pytest.mark.parametrize("C,Hq,Hkv,D,Tp", [
    (42, 8, 1, 64, 20000), (24, 16, 2, 64, 1000), (13, 32, 4, 64, 4096), (40, 8, 1, 128, 9000), (20, 16, 4, 128, 1100),
    (160, 2, 2, 128, 2000), (48, 8, 1, 256, 700), (48, 8, 2, 256, 4096), (33, 16, 8, 256, 769)])
def test_error_is_not_above_the_general_routes(C, Hq, Hkv, D, Tp):
    """Both routes round in fp32; their errors against 64 bits (2-norm over the
    call, some 2e-7 to 3e-7) are roundings of sums whose chains are as short
    here as there: 0.80 to 0.97 of the general route's with chunks of 256 keys.
    A chain over a whole chunk, or operands of fewer bits, is well above 1.1."""
    w = _w(C, Hq, Hkv, D, Tp, (Tp // 8, Tp - Tp // 16), DONOR_DIFF)
    lw = workloads.cell_lw(w)
    bufs = gc.gpu_layer(w, 2)
    q = workloads.make_q(w, 2, 5, device="cuda")
    gc.announce(f"wide f32 error C={C} Hq={Hq} Hkv={Hkv} D={D} Tp={Tp}")
    out, _ = gc.run_attn(w, 2, 5, bufs, q, lw)
    general, _ = gc.run_attn(w, 2, 5, bufs, q, lw, split=max(256, (Tp // 40 + 63) // 64 * 64))
    ref, _ = gc.run_oracle(w, 2, 5, gc.host(bufs), workloads.to_numpy(q), lw)
    err, err_g = (float(np.linalg.norm(x - ref)) for x in (out, general))
    assert err <= 1.1 * err_g, (err / np.linalg.norm(ref), err_g / np.linalg.norm(ref))
    assert np.abs(out - ref).max() <= 4e-6 * np.abs(ref).max()


def test_a_workspace_shared_with_more_cells():
    """The route keeps no counters and leaves its partial results behind those of
    any cell count: a bf16 call with more cells may follow in the same workspace."""
    few = _w(64, 32, 8, 128, 400, (40, 380), DONOR_BLANK)
    many = few.with_(cells=tuple((i % 5, i % 3) for i in range(128)), prompt_len=1100, span=(40, 1000), dtype="bf16")
    need = [sp.splice_decode_attn_workspace_bytes(gc.shape_of(w), sp.make_call(2, 5, 0, w.scale)) for w in (few, many)]
    ws = torch.empty(max(need), dtype=torch.uint8, device="cuda")
    sp.splice_workspace_init(ws)
    for w in (few, many):
        lw = workloads.cell_lw(w)
        bufs = gc.gpu_layer(w, 2)
        q = workloads.make_q(w, 2, 5, device="cuda")
        gc.announce(f"shared workspace {w.dtype} {w.n_cells} cells")
        o, l = gc.run_attn(w, 2, 5, bufs, q, lw, ws=ws)
        o2, l2 = gc.run_attn(w, 2, 5, bufs, q, lw)
        assert np.array_equal(o, o2) and np.array_equal(l, l2), w.dtype
