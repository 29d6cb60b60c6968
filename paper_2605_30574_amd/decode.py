"""Greedy decode of a sweep around the spliced attention (Algorithm 1 of the
paper: per decode step one forward pass, which appends the step's K/V to the
generated cache and attends, then the argmax token; a trajectory stops at
EOS or T_max).

The decoder is a stand-in with synthetic weights (``workloads.model``):
pre-norm blocks of grouped-query attention and a gated MLP.  Per layer and
step the attention -- the current token's K/V appended to each cell's
generated cache, then single-query attention over the cell's spliced prompt
and its generated rows -- is one ``splice_decode_step`` launch of this
library's kernel. Around it, with dense bf16 weights on the GPU, what lies
between the products, the head, the argmax and the products it has better
tiles for are this library's kernels too (``include/splice_decoder.h``); the
other products, and passes with other weights, are PyTorch operations.

Readings of what the paper leaves to the model (the same on the CPU
reference in ``oracle.decoder``):
  * RMSNorm x / sqrt(mean(x^2) + eps) * gain; residual stream in float32;
  * rotary embedding on q and k, pairs (i, i + D/2), angle
    pos * theta^(-2i/D), position T_p + s for decode step s;
  * MLP down(silu(gate(h)) * up(h)); logits from the final norm;
  * the next token is the lowest index of the maximal logit; a cell that
    emits EOS stops (its step becomes -1) and is skipped from then on.
"""
from __future__ import annotations

import ctypes
from typing import List, Optional

import numpy as np
import torch
from torch.autograd import forward_ad
from torch.utils._device import DeviceContext

from . import splice as S

ARGMAX_PARTS = 64   # SPLICE_ARGMAX_PARTS
_declared = None


def _library():
    """The library with the prototypes of include/splice_decoder.h."""
    global _declared
    lib = S.load_library()
    if _declared is not lib:
        vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
        for name, args in (("residual", [vp, vp, vp, i64, i32, vp]),
                           ("norm", [vp, vp, vp, vp, i32, i32, ctypes.c_float, i32, vp]),
                           ("add_norm", [vp, vp, vp, vp, vp, i32, i32, ctypes.c_float, i32, vp]),
                           ("rope_table", [vp, vp, vp, i32, i32, i32, ctypes.c_double, vp]),
                           ("rope", [vp, vp, vp, i32, i32, i32, i32, vp]),
                           ("round", [vp, vp, i32, i32, i32, vp]),
                           ("silu", [vp, vp, vp, i32, i32, i32, vp]), ("product_takes", [i32, i32, i32]), ("head_takes", [i32, i32, i32]),
                           ("product", [vp, vp, vp, i32, i32, i32, vp]),
                           ("head", [vp, vp, vp, i32, i32, i32, vp, ctypes.c_size_t, vp]), ("argmax", [vp, i32, i32, vp, vp, vp])):
            f = getattr(lib, "splice_decoder_" + name)
            f.restype, f.argtypes = i32, args
        lib.splice_decoder_head_bytes.restype, lib.splice_decoder_head_bytes.argtypes = i64, [i32, i32, i32]
        _declared = lib
    return lib


def _unwatched() -> bool:
    """Whether nothing follows the operations of a pass but autograd's backward graph (see _plain): no function
    transform (vmap, jvp, ...), no forward-mode level, no tracer and no mode that sees each operation."""
    return not (torch._C._are_functorch_transforms_active() or forward_ad._current_level >= 0 or
                torch._C._len_torch_dispatch_stack() > 0 or torch._C._get_tracing_state() is not None or
                torch.compiler.is_compiling() or
                any(type(m) is not DeviceContext for m in torch.overrides._get_current_function_mode_stack()))


def _plain(t, device, *shape) -> bool:
    """A bf16 matrix of this shape on the device that autograd does not follow (any strides)."""
    return (type(t) in (torch.Tensor, torch.nn.Parameter) and t.dtype == torch.bfloat16 and t.device == device and
            t.layout == torch.strided and tuple(t.shape) == shape and not (t.requires_grad and torch.is_grad_enabled()))


def _columns(t) -> int:
    """Columns of a weight that is a matrix, else 0 (an object that only knows how to be multiplied, say)."""
    return t.shape[1] if isinstance(t, torch.Tensor) and t.dim() == 2 else 0


def _dense(t) -> bool:
    return t.is_contiguous() and t.data_ptr() % 16 == 0


def _current(device) -> bool:
    """Whether kernels are launched on this GPU: a launch goes to the current device, an operation to its tensors'."""
    return device.index == torch.cuda.current_device()


def greedy(logits: torch.Tensor) -> torch.Tensor:
    """The lowest index of the largest logit of every row (int64)."""
    if not (type(logits) is torch.Tensor and _unwatched() and logits.is_cuda and _current(logits.device) and
            logits.dim() == 2 and logits.is_contiguous() and logits.dtype == torch.float32 and
            0 < logits.shape[0] <= 65535 and 0 < logits.shape[1] <= 1 << 24):
        return torch.argmax(logits, dim=-1)
    n, vocab = logits.shape
    tokens = torch.empty(n, dtype=torch.int64, device=logits.device)
    keys = torch.empty(n * ARGMAX_PARTS, dtype=torch.int64, device=logits.device)
    S._check(_library().splice_decoder_argmax(logits.data_ptr(), n, vocab, tokens.data_ptr(), keys.data_ptr(),
                                              S._stream_ptr(None, logits.device)), "splice_decoder_argmax")
    return tokens


def rms_norm(x: torch.Tensor, gain: torch.Tensor, eps: float) -> torch.Tensor:
    xf = x.float()
    return xf * torch.rsqrt(xf.pow(2).mean(-1, keepdim=True) + eps) * gain.float()


def rope(x: torch.Tensor, pos: torch.Tensor, theta: float) -> torch.Tensor:
    """x [C][H][D] float32, pos [C]: rotate pairs (i, i + D/2) by pos * theta^(-2i/D)."""
    D = x.shape[-1]
    half = D // 2
    inv = theta ** (-torch.arange(0, half, device=x.device, dtype=torch.float64) * 2.0 / D)
    ang = (pos.to(torch.float64)[:, None] * inv[None, :]).to(torch.float32)   # [C][D/2]
    cos, sin = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * cos - x2 * sin, x2 * cos + x1 * sin], dim=-1)


class SweepDecoder:
    """C sweep cells (L_c, W_c) decoding over one prompt, all N layers.

    ``weights`` as drawn by ``workloads.model.make_weights`` (on the device);
    ``caches[l]``: dict clean_k, clean_v, donor_k, donor_v (prompt caches of
    layer l, shared by the cells) and gen_k, gen_v ([C][Hkv][S][D], rows
    written by the decode itself)."""

    def __init__(self, w, m, weights, caches: List[dict], cell_LW, device="cuda"):
        self.w, self.m, self.wt, self.caches = w, m, weights, caches
        self.lw = np.ascontiguousarray(np.asarray(cell_LW, dtype=np.int32).reshape(-1, 2))
        C = self.lw.shape[0]
        self.C, self.N = C, len(weights["layers"])
        self.shape = S.make_shape(C, self.N, w.n_q_heads, w.n_kv_heads, w.head_dim, w.prompt_len, w.span,
                                  w.n_steps, w.donor == "zero", "bf16")
        self.ws = S.new_workspace(self.shape, device=device)
        self.out = torch.empty((C, w.n_q_heads, w.head_dim), dtype=torch.float32, device=device)
        self.lse = torch.empty((C, w.n_q_heads), dtype=torch.float32, device=device)
        self.calls = [S.make_call(l, 0, w.window(l), w.head_dim ** -0.5) for l in range(self.N)]
        self.device = device

    def positions(self, steps: np.ndarray) -> torch.Tensor:
        """Device positions T_p + s of the cells' current tokens."""
        return torch.as_tensor(self.w.prompt_len + np.maximum(steps, 0), device=self.device)

    def forward(self, tokens: torch.Tensor, steps: np.ndarray, pos: Optional[torch.Tensor] = None) -> torch.Tensor:
        """Logits [C][V] (float32) of one decode pass; steps[c] < 0: finished.
        pos: the device positions (self.positions(steps)), given when the pass
        is captured in a graph."""
        w, m, wt = self.w, self.m, self.wt
        C, Hq, Hkv, D = self.C, w.n_q_heads, w.n_kv_heads, w.head_dim
        cdt = wt["embed"].dtype
        x = wt["embed"][tokens]
        if pos is None and getattr(self.positions, "__func__", None) is not SweepDecoder.positions:
            pos = self.positions(steps)   # not the T_p + s that the kernels compute
        if self._fused(x, pos):
            return self._forward_fused(x, steps, pos)
        x = x.float()
        if pos is None:
            pos = self.positions(steps)
        for l in range(self.N):
            p = wt["layers"][l]
            h = rms_norm(x, p["norm_1"], m.rms_eps).to(cdt)
            q = rope((h @ p["w_q"]).float().view(C, Hq, D), pos, m.rope_theta)
            k = rope((h @ p["w_k"]).float().view(C, Hkv, D), pos, m.rope_theta)
            v = (h @ p["w_v"]).float().view(C, Hkv, D)
            c = self.caches[l]
            S.splice_decode_step(self.shape, self.calls[l], self.lw, steps,
                                 q.to(torch.bfloat16).contiguous(), k.to(torch.bfloat16).contiguous(),
                                 v.to(torch.bfloat16).contiguous(), c["clean_k"], c["clean_v"], c["donor_k"],
                                 c["donor_v"], c["gen_k"], c["gen_v"], self.out, self.lse, self.ws)
            x = x + (self.out.view(C, Hq * D).to(cdt) @ p["w_o"]).float()
            h = rms_norm(x, p["norm_2"], m.rms_eps).to(cdt)
            x = x + ((torch.nn.functional.silu((h @ p["w_gate"]).float()).to(cdt) * (h @ p["w_up"]))
                     @ p["w_down"]).float()
        return (rms_norm(x, wt["norm_f"], m.rms_eps).to(cdt) @ wt["lm_head"]).float()

    def _fused(self, x: torch.Tensor, pos: Optional[torch.Tensor]) -> bool:
        """Whether the library's kernels take this pass (x: the embedded tokens)."""
        w, wt = self.w, self.wt
        C, Hq, Hkv, D, dev, d = self.C, w.n_q_heads, w.n_kv_heads, w.head_dim, x.device, x.shape[-1]
        if torch.is_autocast_enabled("cuda") and torch.get_autocast_dtype("cuda") != torch.bfloat16:
            return False   # the products are another type's
        if not (_unwatched() and x.is_cuda and _current(dev) and C > 0 and d % 8 == 0 and _plain(x, dev, C, d) and
                _dense(x) and (pos is None or (pos.device == dev and tuple(pos.shape) == (C,)))):
            return False
        for p in wt["layers"]:
            F = _columns(p["w_gate"])
            if not (F % 8 == 0 and F > 0 and _plain(p["w_gate"], dev, d, F) and _plain(p["w_up"], dev, d, F) and
                    _plain(p["w_down"], dev, F, d) and _plain(p["w_q"], dev, d, Hq * D) and
                    _plain(p["w_k"], dev, d, Hkv * D) and _plain(p["w_v"], dev, d, Hkv * D) and
                    _plain(p["w_o"], dev, Hq * D, d) and _plain(p["norm_1"], dev, d) and _dense(p["norm_1"]) and
                    _plain(p["norm_2"], dev, d) and _dense(p["norm_2"])):
                return False
        head = wt["lm_head"]
        return _plain(wt["norm_f"], dev, d) and _dense(wt["norm_f"]) and _plain(head, dev, d, _columns(head))

    def _forward_fused(self, delta: torch.Tensor, steps, pos: Optional[torch.Tensor]) -> torch.Tensor:
        """forward() with the library's kernels between the products: the same roundings, so the same bits up to the head."""
        w, m, wt, lib = self.w, self.m, self.wt, _library()
        C, Hq, Hkv, D, d, dev = self.C, w.n_q_heads, w.n_kv_heads, w.head_dim, delta.shape[1], delta.device
        bf16, stream = torch.bfloat16, S._stream_ptr(None, delta.device)
        ok = S._check
        # one kernel a norm where it adds in the order of mean(), so that the
        # bits stay: fewer rows, shorter and longer ones are added in others
        # (measured: 8184 values differ, 7680 do not)
        one_norm = C >= 8 and 256 <= d <= 7680
        x = torch.empty((C, d), dtype=torch.float32, device=dev)   # the residual stream
        sq = None if one_norm else torch.empty_like(x)
        h = torch.empty(((C + 15) // 16 * 16, d), dtype=bf16, device=dev)[:C]
        o = torch.empty((C, Hq * D), dtype=bf16, device=dev)
        tab = torch.empty((C, D), dtype=torch.float32, device=dev)
        xp, hp, op, tp, outp = (t.data_ptr() for t in (x, h, o, tab, self.out))
        st, stp = S._steps(steps, C)
        if pos is not None:
            pos = pos.to(torch.float64).contiguous()
        ok(lib.splice_decoder_rope_table(tp, None if pos is None else pos.data_ptr(), stp, C, D, w.prompt_len,
                                         float(m.rope_theta), stream), "splice_decoder_rope_table")

        def norm(delta, gain, assign=0, packed=0):
            """x += delta (the first: x = delta); h = bf16(rms_norm(x)), packed for the head (2: both, packed in hq)."""
            if one_norm:
                ok(lib.splice_decoder_add_norm(xp, delta.data_ptr(), gain.data_ptr(), None if packed == 1 else hp,
                                               (None, hp, hqp)[packed], C, d, m.rms_eps, assign, stream),
                   "splice_decoder_add_norm")
                return
            ok(lib.splice_decoder_residual(xp, delta.data_ptr(), sq.data_ptr(), C * d, assign, stream),
               "splice_decoder_residual")
            mean = sq.mean(-1, keepdim=True)
            ok(lib.splice_decoder_norm(xp, mean.data_ptr(), gain.data_ptr(), hp, C, d, m.rms_eps, packed, stream),
               "splice_decoder_norm")

        def own(w):
            """Whether the library's own product takes this weight."""
            return one_norm and _dense(w) and lib.splice_decoder_product_takes(C, w.shape[0], w.shape[1]) == 1

        def product(x_packed, w):
            y = torch.empty((C, w.shape[1]), dtype=bf16, device=dev)
            ok(lib.splice_decoder_product(x_packed, w.data_ptr(), y.data_ptr(), C, w.shape[0], w.shape[1], stream),
               "splice_decoder_product")
            return y

        hq = torch.empty_like(h) if any(own(p["w_q"]) for p in wt["layers"]) else h
        hqp = hq.data_ptr()
        first = 1
        for l in range(self.N):
            p, c = wt["layers"][l], self.caches[l]
            own_q, own_o, own_down = own(p["w_q"]), own(p["w_o"]), own(p["w_down"])
            norm(delta, p["norm_1"], first, 2 if own_q else 0)
            first = 0
            q = product(hqp, p["w_q"]) if own_q else h @ p["w_q"]
            k, v = h @ p["w_k"], h @ p["w_v"]
            ok(lib.splice_decoder_rope(q.data_ptr(), k.data_ptr(), tp, C, Hq, Hkv, D, stream), "splice_decoder_rope")
            S.splice_decode_step(self.shape, self.calls[l], self.lw, st, q, k, v, c["clean_k"], c["clean_v"],
                                 c["donor_k"], c["donor_v"], c["gen_k"], c["gen_v"], self.out, self.lse, self.ws)
            ok(lib.splice_decoder_round(outp, op, C, Hq * D, own_o, stream), "splice_decoder_round")
            norm(product(op, p["w_o"]) if own_o else o @ p["w_o"], p["norm_2"])
            gate, up = h @ p["w_gate"], h @ p["w_up"]
            act = torch.empty_like(gate) if own_down else gate
            ok(lib.splice_decoder_silu(gate.data_ptr(), up.data_ptr(), act.data_ptr(), C, gate.shape[1], own_down, stream),
               "splice_decoder_silu")
            delta = product(act.data_ptr(), p["w_down"]) if own_down else act @ p["w_down"]
        head = wt["lm_head"]
        vocab = head.shape[1]
        own_head = _dense(head) and lib.splice_decoder_head_takes(C, d, vocab) == 1
        norm(delta, wt["norm_f"], first, own_head)
        if not own_head:
            return (h @ head).float()
        logits = torch.empty((C, vocab), dtype=torch.float32, device=dev)
        need = ok(lib.splice_decoder_head_bytes(C, d, vocab), "splice_decoder_head_bytes")
        part = torch.empty(need, dtype=torch.uint8, device=dev)
        ok(lib.splice_decoder_head(hp, head.data_ptr(), logits.data_ptr(), C, d, vocab, part.data_ptr(), need, stream),
           "splice_decoder_head")
        return logits

    def step(self, tokens: torch.Tensor, steps: np.ndarray, pos: Optional[torch.Tensor] = None):
        """One decode pass: (next tokens [C] int64, logits [C][V]); of equal
        largest logits the lowest index."""
        logits = self.forward(tokens, steps, pos)
        return greedy(logits), logits


def advance(steps: np.ndarray, next_tokens: np.ndarray, eos: int, n_steps: int) -> np.ndarray:
    """The cells' steps after a pass: +1, or -1 for a cell that emitted EOS or
    reached T_max (= the generated-cache capacity)."""
    s = steps.copy()
    act = s >= 0
    s[act] += 1
    s[act & (next_tokens == eos)] = -1
    s[s >= n_steps] = -1
    return s
