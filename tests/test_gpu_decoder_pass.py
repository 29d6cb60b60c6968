"""The fused decode pass (bf16 weights: this library's kernels between the
products) against the same pass written out in PyTorch operations.

The fused kernels round where the operations they replace round, so what
enters and leaves every product is the same bit for bit: the appended cache
rows are equal.  The head is the library's own product: the same bf16 inputs
summed in fp32 in another order, then rounded to bf16 as the operation's
output is, so a logit differs by at most one bf16 step (2^-7 of its size) plus
both sums' own error, d 2^-24 times the sum of |h w| at most.  |h| is about 1
and |w| about d^-1/2, so that sum is below 8 sqrt(d)."""
import types

import numpy as np
import pytest
import torch
from torch.autograd import forward_ad

import gpu_common as gc
import paper_2605_30574_amd as sp
import workloads
from paper_2605_30574_amd import decode
from workloads.model import ModelConfig, make_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    sp.load_library()


def _decoder(C, d, F, V, Hq, Hkv, D, N, seed=0):
    w = workloads.get(1).with_(n_layers=N, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=D, prompt_len=40, span=(5, 33),
                               n_steps=16, cells=tuple((i % (N + 1), i % 4) for i in range(C)), scale=D ** -0.5)
    m = ModelConfig(d_model=d, d_ff=F, vocab=V, eos=0)
    wt = make_weights(w, m, seed=seed, dtype=torch.bfloat16, device="cuda", draw_on_device=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    for L in wt["layers"]:
        for n in ("norm_1", "norm_2"):
            L[n] = (1 + 0.2 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    wt["norm_f"] = (1 + 0.2 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    lw = workloads.cell_lw(w)

    def make(fused):
        dec = decode.SweepDecoder(w, m, wt, [gc.gpu_layer(w, l) for l in range(N)], lw)
        if not fused:
            dec._fused = lambda *a: False
        return dec
    rng = np.random.default_rng(seed)
    steps = rng.integers(0, w.n_steps, size=C).astype(np.int32)
    tokens = torch.as_tensor(rng.integers(0, V, size=C), device="cuda")
    return make, wt, tokens, steps


def _compare(make, wt, tokens, steps, what, pos=None):
    gc.announce(f"decoder pass {what}")
    a, b = make(True), make(False)
    assert a._fused(wt["embed"][tokens], pos), "the fused path did not take the pass"
    tok, got = a.step(tokens, steps, pos)
    want = b.forward(tokens, steps, pos)
    torch.cuda.synchronize()
    for ca, cb in zip(a.caches, b.caches):
        for n in ("gen_k", "gen_v"):
            assert torch.equal(ca[n].view(torch.int16), cb[n].view(torch.int16)), f"{what}: {n}"
    d = wt["lm_head"].shape[0]
    bound = 2.0 ** -7 * want.abs() + 2 * d * 2.0 ** -24 * 8 * d ** 0.5
    assert torch.isfinite(got).all() and ((got - want).abs() <= bound).all(), what
    assert torch.equal(tok, torch.argmax(got, -1)), what


# rows around the head's row blocks, the smallest sizes, K and vocabulary with
# partial column tiles, columns split over K in the last round (vocabulary 66600)
@pytest.mark.parametrize("C,d,F,V,Hq,Hkv,D,N", [
    (1, 32, 32, 8, 2, 1, 64, 1), (16, 96, 160, 136, 4, 2, 64, 2), (17, 256, 416, 1000, 8, 2, 64, 1),
    (33, 320, 96, 264, 4, 4, 128, 2), (65, 128, 512, 520, 4, 2, 256, 1), (128, 512, 768, 4104, 8, 8, 64, 1),
    (129, 224, 352, 264, 4, 2, 64, 1), (256, 256, 64, 512, 2, 1, 64, 1), (24, 1056, 64, 66600, 2, 1, 64, 1),
    (100, 1056, 64, 66600, 2, 1, 64, 1), (64, 2048, 256, 264, 32, 4, 64, 1), (128, 2056, 2176, 264, 16, 2, 128, 2), (9, 72, 104, 100, 4, 2, 64, 1),
    # the second layer's cache rows follow the first one's products: the query, output and down projections the
    # library's own kernel takes, and the 2048 columns at 128 rows it leaves
    # more rows than one pass over the head's weights, and a long K for few columns: the library's head
    (130, 256, 64, 49160, 2, 1, 64, 1), (20, 2304, 64, 264, 2, 1, 64, 1),
    (64, 2048, 2176, 264, 32, 4, 64, 2), (128, 2560, 2176, 264, 32, 8, 128, 2), (128, 2048, 2176, 264, 32, 4, 64, 2)])
def test_fused_pass_keeps_the_bits(C, d, F, V, Hq, Hkv, D, N):
    make, wt, tokens, steps = _decoder(C, d, F, V, Hq, Hkv, D, N)
    _compare(make, wt, tokens, steps, f"C={C} d={d} F={F} V={V} D={D}")


def test_given_positions_finished_cells_and_strided_weights():
    make, wt, tokens, steps = _decoder(20, 96, 160, 136, 4, 2, 64, 2)
    for pos in (torch.arange(20, device="cuda") * 37, torch.arange(20, device="cuda").float() * 411.0):
        _compare(make, wt, tokens, steps, f"positions {pos.dtype}", pos)
    done = steps.copy()
    done[3] = done[11] = -1   # their attention rows are not written: keep them finite in both
    a, b = make(True), make(False)
    a.out.zero_()
    b.out.zero_()
    got, want = a.forward(tokens, done), b.forward(tokens, done)
    assert torch.allclose(got, want, rtol=2 ** -7, atol=1e-3)
    for n in ("w_q", "w_down"):   # a transposed view is taken as it is
        for L in wt["layers"]:
            L[n] = L[n].t().contiguous().t()
    wt["lm_head"] = wt["lm_head"].t().contiguous().t()
    _compare(make, wt, tokens, steps, "strided weights")


def test_overridden_positions_are_used():
    make, wt, tokens, steps = _decoder(9, 96, 160, 136, 4, 2, 64, 1)
    got = []
    for given in (False, True):
        dec = make(True)
        far = dec.positions(steps) + 1000
        if not given:
            dec.positions = lambda s: far
        gc.announce(f"decoder pass, positions given={given}")
        got.append((dec.forward(tokens, steps, far if given else None), dec.caches[0]["gen_k"]))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


class _Product:
    """A weight that is no tensor: h @ weight is all it knows."""

    def __init__(self, w):
        self.w = w

    def __rmatmul__(self, h):
        return h @ self.w


def test_weights_that_only_multiply():
    make, wt, tokens, steps = _decoder(5, 96, 160, 136, 4, 2, 64, 1)
    want = make(False).forward(tokens, steps)
    for owner, name in ((wt["layers"][0], "w_gate"), (wt["layers"][0], "w_q"), (wt, "lm_head")):
        keep, owner[name] = owner[name], _Product(owner[name])
        gc.announce(f"decoder pass, {name} an object")
        got = make(True).forward(tokens, steps)
        owner[name] = keep
        assert torch.equal(got, want), name


def test_another_current_device_keeps_the_operations(monkeypatch):
    make, wt, tokens, steps = _decoder(5, 96, 160, 136, 4, 2, 64, 1)
    x = wt["embed"][tokens]
    assert make(True)._fused(x, None)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: x.device.index + 1)
    assert not make(True)._fused(x, None)
    monkeypatch.setattr(decode, "_library", None)   # greedy() would call it
    assert decode.greedy(x.float()).shape == (5,)


def test_other_weights_take_the_written_out_pass():
    make, wt, tokens, steps = _decoder(5, 96, 160, 136, 4, 2, 64, 1)
    dec = make(True)
    x = wt["embed"][tokens]
    assert dec._fused(x, None)
    keep = wt["layers"][0]["norm_1"]
    for bad in (keep.float(), torch.stack([keep, keep], 1)[:, 0]):   # another type, a strided gain
        wt["layers"][0]["norm_1"] = bad
        assert not dec._fused(x, None)
        dec.forward(tokens, steps)
    wt["layers"][0]["norm_1"] = keep.clone().requires_grad_()
    assert not dec._fused(x, None)
    with torch.no_grad():
        assert dec._fused(x, None)
    wt["layers"][0]["norm_1"] = keep
    assert not dec._fused(x.float(), None) and not dec._fused(x, torch.arange(5))
    elsewhere = types.SimpleNamespace(is_cuda=True, shape=(5,), device=torch.device("cuda", x.device.index + 1))
    assert not dec._fused(x, elsewhere)   # the operation refuses positions on another GPU


def test_transforms_and_forward_mode_see_the_head():
    """A dual or transformed head's product is the operation, which carries the tangent (and the batch)."""
    make, wt, tokens, steps = _decoder(6, 96, 160, 136, 4, 2, 64, 1)
    head, tan = wt["lm_head"], torch.randn_like(wt["lm_head"])
    fused = make(True)

    def logits(w):
        wt["lm_head"] = w
        try:
            return fused.forward(tokens, steps)
        finally:
            wt["lm_head"] = head

    gc.announce("decoder pass under vmap and forward mode")
    with torch.no_grad():
        dec = make(False)
        want = dec.forward(tokens, steps)
        wt["lm_head"] = tan
        want_tan = make(False).forward(tokens, steps)   # the logits are linear in the head
        wt["lm_head"] = head
    with forward_ad.dual_level():
        got = forward_ad.unpack_dual(logits(forward_ad.make_dual(head, tan)))
        assert torch.equal(got.primal, want) and torch.equal(got.tangent, want_tan)
    both = torch.vmap(lambda w: logits(w))(torch.stack([head, tan]))
    assert torch.allclose(both, torch.stack([want, want_tan]), rtol=2 ** -7, atol=1e-3)
    toks = torch.vmap(decode.greedy)(torch.stack([want, want_tan]))
    assert torch.equal(toks, torch.argmax(torch.stack([want, want_tan]), -1))


def test_autocast_passes():
    make, wt, tokens, steps = _decoder(6, 96, 160, 136, 4, 2, 64, 1)
    for dtype in (torch.float16, torch.bfloat16):
        with torch.autocast("cuda", dtype):
            gc.announce(f"decoder pass under autocast {dtype}")
            a, b = make(True), make(False)
            assert a._fused(wt["embed"][tokens], None) == (dtype == torch.bfloat16)
            got, want = a.forward(tokens, steps), b.forward(tokens, steps)
        assert torch.allclose(got, want, rtol=2 ** -7, atol=1e-3)
        for n in ("gen_k", "gen_v"):
            assert torch.equal(a.caches[0][n], b.caches[0][n])


def test_norm_rounds_as_the_operations():
    g = torch.Generator(device="cuda").manual_seed(3)
    C, d, lib = 256, 1024, decode._library()
    buf = torch.empty(2, C, d, device="cuda")
    for scale in (1e-3, 1.0, 300.0):
        x, delta = torch.randn(C, d, generator=g, device="cuda") * scale, torch.randn(C, d, generator=g, device="cuda").bfloat16()
        gain = (1 + 0.2 * torch.randn(d, generator=g, device="cuda")).bfloat16()
        h = torch.empty(C, d, device="cuda", dtype=torch.bfloat16)
        buf[0].copy_(x)
        gc.announce(f"norm scale {scale}")
        assert lib.splice_decoder_residual(buf[0].data_ptr(), delta.data_ptr(), buf[1].data_ptr(), C * d, 0, None) == 0
        mean = buf[1].mean(-1, keepdim=True)
        assert lib.splice_decoder_norm(buf[0].data_ptr(), mean.data_ptr(), gain.data_ptr(), h.data_ptr(), C, d, 1e-6, 0,
                                       None) == 0
        assert torch.equal(buf[0], x + delta.float())
        assert torch.equal(h, decode.rms_norm(x + delta.float(), gain, 1e-6).bfloat16())


# the smallest and largest sizes the pass takes it at, units that fill the last
# round in part, and sizes beyond, which it does not take: there the operation
# adds in another order and the mean differs by a few ulp
@pytest.mark.parametrize("C,d", [(8, 256), (9, 264), (128, 1032), (8, 2560), (130, 4096), (256, 7680), (8, 7672), (1, 8), (3, 8192),
                                 (256, 8184)])
def test_add_norm_adds_as_the_mean(C, d):
    g = torch.Generator(device="cuda").manual_seed(d)
    x, delta = torch.randn(C, d, generator=g, device="cuda"), torch.randn(C, d, generator=g, device="cuda").bfloat16()
    gain = (1 + 0.2 * torch.randn(d, generator=g, device="cuda")).bfloat16()
    lib = decode._library()
    for assign in (0, 1):
        want_x = delta.float() if assign else x + delta.float()
        want = decode.rms_norm(want_x, gain, 1e-6).bfloat16()
        for packed in (0, 1) if d % 32 == 0 else (0,):
            rows = (C + 15) // 16 * 16
            y, h = x.clone(), torch.zeros(rows, d, device="cuda", dtype=torch.bfloat16)
            gc.announce(f"add_norm {C}x{d} assign={assign} packed={packed}")
            assert lib.splice_decoder_add_norm(y.data_ptr(), delta.data_ptr(), gain.data_ptr(), None if packed else h.data_ptr(),
                                               h.data_ptr() if packed else None, C, d, 1e-6, assign, None) == 0
            got = h.view(d // 32, rows // 16, 16, 32).permute(1, 2, 0, 3).reshape(rows, d) if packed else h
            assert torch.equal(y, want_x)
            if C >= 8 and 256 <= d <= 7680:
                assert torch.equal(got[:C], want)
            else:   # another order of the sum: one bf16 step at most
                assert ((got[:C].float() - want.float()).abs() <= 2.0 ** -7 * want.float().abs()).all()
            assert not got[C:].any()
    assert lib.splice_decoder_add_norm(x.data_ptr(), delta.data_ptr(), gain.data_ptr(), h.data_ptr(), None, C, 8200, 1e-6, 0,
                                       None) == sp.SPLICE_EUNSUPPORTED


def test_head_takes():
    takes = decode._library().splice_decoder_head_takes
    for dims, want in (((128, 4096, 151936), 1), ((129, 4096, 151936), 0), ((128, 4096, 49152), 1), ((128, 4096, 32000), 0),
                       ((16, 4096, 16384), 1), ((16, 5120, 16384), 0), ((64, 2048, 264), 1), ((64, 2080, 264), 0),
                       ((128, 1024, 264), 1), ((128, 1056, 264), 0), ((200, 1024, 264), 1), ((8, 2560, 151936), 1),
                       ((8, 2568, 151936), 0), ((8, 2560, 151940), 0)):
        assert takes(*dims) == want, dims


# one and several row groups, rows and columns that fill the last tile in part,
# K of one stage, of fewer stages than the ring and of many
@pytest.mark.parametrize("rows,K,N", [(1, 128, 8), (33, 256, 72), (64, 512, 2048), (128, 4096, 2056), (200, 1408, 136)])
def test_product(rows, K, N):
    g = torch.Generator(device="cuda").manual_seed(K + N)
    x = torch.randn(rows, K, generator=g, device="cuda").bfloat16()
    w = (torch.randn(K, N, generator=g, device="cuda") * K ** -0.5).bfloat16()
    pad = (rows + 15) // 16 * 16
    xp = torch.zeros(pad, K, device="cuda", dtype=torch.bfloat16)
    xp[:rows] = x
    xp = xp.view(pad // 16, 16, K // 32, 32).permute(2, 0, 1, 3).contiguous()
    y = torch.full((rows + 1, N), 7.0, device="cuda", dtype=torch.bfloat16)
    gc.announce(f"product {rows}x{K}x{N}")
    lib = decode._library()
    assert lib.splice_decoder_product(xp.data_ptr(), w.data_ptr(), y.data_ptr(), rows, K, N, None) == 0
    want = (x.double() @ w.double())
    bound = 2.0 ** -8 * want.abs() + K * 2.0 ** -24 * (x.double().abs() @ w.double().abs())   # rounding, fp32 sums
    assert ((y[:rows].double() - want).abs() <= bound).all() and (y[rows] == 7).all()
    assert lib.splice_decoder_product(xp.data_ptr(), w.data_ptr(), y.data_ptr(), rows, K + 32, N, None) == sp.SPLICE_EUNSUPPORTED


# the sizes of the models' projections, the smallest and largest K, columns that
# fill the last tile in part: where a pass takes the own product, its bits are
# those of the operation it replaces
@pytest.mark.parametrize("rows", [64, 128])
@pytest.mark.parametrize("K", [128, 1408, 2048, 2560, 4096, 8192, 9728, 12288, 14336, 16384])
def test_product_has_the_operations_bits(rows, K):
    g = torch.Generator(device="cuda").manual_seed(K + rows)
    lib = decode._library()
    x = torch.randn(rows, K, generator=g, device="cuda").bfloat16()
    xp = x.view(rows // 16, 16, K // 32, 32).permute(2, 0, 1, 3).contiguous()
    for N in (2048, 2056, 2560, 3080, 4000, 4096, 5120, 8192):
        takes = lib.splice_decoder_product_takes(rows, K, N) == 1
        assert takes == (N <= 4096 and N > 2048 if rows == 128 else True)
        if not takes:
            continue
        w = (torch.randn(K, N, generator=g, device="cuda") * K ** -0.5).bfloat16()
        y = torch.empty(rows, N, device="cuda", dtype=torch.bfloat16)
        gc.announce(f"product bits {rows}x{K}x{N}")
        assert lib.splice_decoder_product(xp.data_ptr(), w.data_ptr(), y.data_ptr(), rows, K, N, None) == 0
        assert torch.equal(y.view(torch.int16), (x @ w).view(torch.int16)), N
    assert lib.splice_decoder_product_takes(rows, 17920, 4096) == 0   # the library splits K there


@pytest.mark.parametrize("rows,vocab", [(1, 1), (3, 257), (130, 1023), (7, 70001)])
def test_greedy_is_argmax(rows, vocab):
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randint(-3, 4, (rows, vocab), generator=g, device="cuda").float()   # many ties
    x[x == 0] = -0.0
    gc.announce(f"greedy {rows}x{vocab}")
    assert torch.equal(decode.greedy(x), torch.argmax(x, -1))
    x[0, :] = float("-inf")
    x[rows // 2, vocab // 2] = float("inf")
    x[rows - 1, vocab - 1] = float("nan")
    x[rows - 1, vocab // 3] = float("nan")
    assert torch.equal(decode.greedy(x), torch.argmax(x, -1))
    assert torch.equal(decode.greedy(x.double()), torch.argmax(x, -1))   # other types: the operation itself
