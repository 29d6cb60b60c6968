"""Merging 8, 9, 16 and 17 prompt slots (the generated-row item's in-place
merge keeps the rows' records in registers up to 8 slots, in LDS up to 16, and
takes rounds beyond): the same bits as the hand-over merge, and the oracle."""
import numpy as np
import pytest
import torch

import gpu_common as gc
import paper_2605_30574_amd as sp
import workloads
from workloads import DONOR_BLANK, DONOR_ZERO

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sp.load_library()


@pytest.mark.parametrize("D,G", [(64, 1), (128, 4), (128, 8), (256, 8)])
@pytest.mark.parametrize("n_slots", [8, 9, 16, 17])
def test_slots(D, G, n_slots):
    Tp = 64 * n_slots - 5
    for donor, step, C in ((DONOR_BLANK, 3, 9), (DONOR_ZERO, 140, 5)):
        w = workloads.get("qwen3-4b").with_(n_layers=4, n_q_heads=2 * G, n_kv_heads=2, head_dim=D, prompt_len=Tp,
                                             span=(33, Tp - 40), n_steps=150, donor=donor, scale=D ** -0.5,
                                             cells=tuple((i % 5, i % 3) for i in range(C)))
        lw = workloads.cell_lw(w)
        bufs = gc.gpu_layer(w, 2)
        q = workloads.make_q(w, 2, step, device="cuda")
        gc.announce(f"merge slots D={D} G={G} n={n_slots} step={step}")
        o, l = gc.run_attn(w, 2, step, bufs, q, lw, split=64)
        oh, lh = gc.run_attn(w, 2, step, bufs, q, lw, split=64, merge_wait=-1)
        assert np.array_equal(o, oh) and np.array_equal(l, lh)
        ref_o, ref_l = gc.run_oracle(w, 2, step, gc.host(bufs), workloads.to_numpy(q), lw)
        gc.assert_attn_close(o, l, ref_o, ref_l, f"{n_slots} slots")
