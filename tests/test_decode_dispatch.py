"""When a decode pass may leave PyTorch's operations (on the CPU: the rule only;
the passes themselves are compared in test_gpu_decoder_pass.py)."""
import contextlib

import torch
from torch.autograd import forward_ad
from torch.fx.experimental.proxy_tensor import make_fx
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2605_30574_amd import decode


class _Dispatch(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


class _Function(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_watchers_keep_the_operations():
    assert decode._unwatched()
    for mode in (forward_ad.dual_level(), _Dispatch(), _Function()):
        with mode:
            assert not decode._unwatched(), mode
    for mode in (torch.no_grad(), torch.inference_mode(), torch.device("cpu"), contextlib.nullcontext()):
        with mode:
            assert decode._unwatched(), mode
    seen = []

    def f(x):
        seen.append(decode._unwatched())
        return x * 2

    one = torch.ones(3)
    torch.func.jvp(f, (one,), (one,))
    torch.vmap(f)(one)
    torch.func.grad(lambda x: f(x).sum())(one)
    make_fx(f)(one)
    torch.jit.trace(f, one, check_trace=False)
    assert seen and not any(seen), seen
    assert decode._unwatched()
