"""The two calls on tensors: the errors that torch raises while they allocate outputs, and what they take for parameters.
A program that catches torch.OutOfMemoryError to free memory and try again has to see that type, as from torch.empty itself."""
import ctypes

import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2002_11082_amd as ogq


class RefuseToAllocate(TorchDispatchMode):
    """Every allocation raises `error`; nothing else is touched."""

    def __init__(self, error):
        super().__init__()
        self.error = error

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is torch.ops.aten.empty.memory_format:
            raise self.error
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("error", [torch.OutOfMemoryError("no memory left"), NotImplementedError("not here"), KeyError("mine")])
def test_an_error_while_allocating_outputs_keeps_its_type(error):
    """On tensors without memory (no GPU): the allocation is refused before any pointer is taken."""
    n, p = 4096, ogq.make_params(512, 1, ogq.BINGRAD_B)
    with FakeTensorMode():
        grad = torch.empty(n, device="cuda")
        levels = torch.empty(ogq.ogq_levels_count(n, p), device="cuda")
        codes = torch.empty(ogq.ogq_codes_bytes(n, p) // 8, dtype=torch.int64, device="cuda")
    for call in (lambda: ogq.ogq_quantize(grad, p), lambda: ogq.ogq_quantize(grad, p, levels),
                 lambda: ogq.ogq_quantize(grad, p, None, codes), lambda: ogq.ogq_dequantize_average([codes], [levels], n, p)):
        with RefuseToAllocate(error), pytest.raises(type(error)) as caught:
            call()
        assert caught.value is error


class OtherStructure(ctypes.Structure):
    _fields_ = [("words", ctypes.c_uint32 * 10)]


@pytest.mark.parametrize("params", [bytes(40), bytearray(40), OtherStructure(), None, 512],
                         ids=["bytes", "bytearray", "structure", "none", "number"])
def test_only_params_are_taken_for_parameters(params):
    """Forty bytes of anything else were read as a bucket size, a scheme and so on."""
    with FakeTensorMode():
        grad = torch.empty(4096, device="cuda")
        codes = torch.empty(128, dtype=torch.int64, device="cuda")
    with pytest.raises(TypeError):
        ogq.ogq_quantize(grad, params)
    with pytest.raises(TypeError):
        ogq.ogq_dequantize_average([codes], [grad], 4096, params)


@pytest.mark.gpu
def test_out_of_memory_is_torch_out_of_memory():
    """The allocator's own refusal (a limit on this process's share of the memory, nothing is exhausted), and the calls
    work again once it is lifted."""
    dev, n = "cuda:0", 128 << 20
    p = ogq.make_params(2048, 1, ogq.BINGRAD_B)
    grad = torch.randn(n, device=dev)
    levels, codes = ogq.ogq_quantize(grad, p)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    torch.cuda.set_per_process_memory_fraction(1e-6, 0)
    try:
        with pytest.raises(torch.OutOfMemoryError):  # what the allocator still has, in pieces of the smaller output's size
            while True:
                held.append(torch.empty_like(codes))
        with pytest.raises(torch.OutOfMemoryError):
            ogq.ogq_quantize(grad, p, levels)
        with pytest.raises(torch.OutOfMemoryError):
            ogq.ogq_dequantize_average([codes], [levels], n, p)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0, 0)
    again_levels, again_codes = ogq.ogq_quantize(grad, p)
    out = ogq.ogq_dequantize_average([again_codes], [again_levels], n, p)
    torch.cuda.synchronize()
    assert torch.equal(again_levels, levels) and torch.equal(again_codes, codes) and out.numel() == n
