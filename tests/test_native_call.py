"""The binding's native calls: they refuse what the Python checks refuse, and convert numbers as ctypes does."""
import ctypes
import os
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_1804_02941_amd import binding, build


@pytest.fixture(scope="module")
def call():
    if not (os.path.exists(binding.LIB_PATH) and os.path.exists(build.CALL)):
        build.build()
    return binding.native()


def test_every_function_has_the_entry_points_arity(call):
    for name in (n for n in dir(call) if n.startswith("dab_")):
        res, args = binding._SIGNATURES[name]
        n = len(args) - (res is ctypes.c_int)                      # the stream is supplied
        with pytest.raises(TypeError, match=f"takes {n} arguments"):
            getattr(call, name)(*[None] * (n + 1))


def test_sizes_and_numbers(call):
    for case in ((8192, 9216, 512), (4, 100, 4), (0, 100, 4), (True, 64, 64), (2 ** 32 + 8192, 9216, 512), (-1, 64, 64)):
        assert call.dab_binfc_workspace_bytes(*case) == binding.lib().dab_binfc_workspace_bytes(*case)
    d = binding.dab_conv_desc(256, 512, 7, 7, 512, 3, 3, 1, 1, 1, 1)
    assert call.dab_wbin_conv2d_workspace_bytes(d) == binding.lib().dab_wbin_conv2d_workspace_bytes(ctypes.byref(d)) > 0
    for bad in ((1.5, 2, 3), ("1", 2, 3), (None, 2, 3)):
        with pytest.raises(ctypes.ArgumentError):
            call.dab_binfc_workspace_bytes(*bad)
    with pytest.raises(ctypes.ArgumentError):
        call.dab_binconv2d_workspace_bytes(bytes(44))


class Sized:
    _as_parameter_ = 9216


@pytest.mark.parametrize("n", [np.int64(9216), np.int32(9216), np.uint8(64), torch.tensor(9216), torch.tensor([9216]), np.array(9216),
                               ctypes.c_int32(9216), Sized(), np.float32(9216.0), torch.tensor(9216.0), np.array([9216, 1]), 9216j,
                               Fraction(9216)])
def test_numbers_of_other_types_are_taken_and_refused_as_ctypes_does(call, n):
    def result(f, *a):
        try:
            return f(*a)
        except ctypes.ArgumentError:
            return "refused"
    for args in ((8192, n, 512), (n, 9216, 512)):
        assert result(call.dab_binfc_workspace_bytes, *args) == result(binding.lib().dab_binfc_workspace_bytes, *args)


@pytest.mark.gpu
@pytest.mark.parametrize("lo", [np.float32(-0.5), np.float64(-0.5), Fraction(-1, 2), torch.tensor(-0.5), ctypes.c_float(-0.5)])
def test_limits_of_other_types(lo):
    W = torch.randn(4, 3, 3, 3, device="cuda:0")
    ref = binding.dab_mean_center_clamp(W, lo=-0.5, hi=1.0)
    assert torch.equal(binding.dab_mean_center_clamp(W, lo=lo, hi=np.int32(1)), ref)
    with pytest.raises(ctypes.ArgumentError):
        binding.dab_mean_center_clamp(W, lo="-0.5")


@pytest.mark.parametrize("X", [torch.zeros(2, 64), torch.nn.Parameter(torch.zeros(2, 64)), [[0.0] * 64] * 2])
def test_what_is_not_on_the_gpu_is_refused(call, X):
    with pytest.raises(TypeError, match="X: expected a tensor on the GPU"):
        call.dab_pack_activations(X, 0, 2, 64, 1, 1, None, None)


@pytest.mark.gpu
def test_types_strides_and_status(call):
    X = torch.randn(4, 64, device="cuda:0")
    A = torch.empty((4, 1, 1, 2), dtype=torch.int32, device=X.device)
    with pytest.raises(TypeError, match="X: expected torch.float32, got torch.float64"):
        call.dab_pack_activations(X.double(), 0, 4, 64, 1, 1, None, A)
    with pytest.raises(ValueError, match="X: tensor must be contiguous"):
        call.dab_pack_activations(X.t(), 0, 4, 64, 1, 1, None, A)
    with pytest.raises(TypeError, match="A_packed: expected torch.int32"):
        call.dab_pack_activations(X, 0, 4, 64, 1, 1, None, A.long())
    with pytest.raises(binding.DabError, match="dab_pack_activations failed: status 1"):
        call.dab_pack_activations(None, 0, 4, 64, 1, 1, None, A)
    ref = binding.dab_pack_activations(X)
    for form in (X, torch.nn.Parameter(X, requires_grad=False)):
        assert torch.equal(binding.dab_pack_activations(form), ref)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):                                   # the call goes to the current stream
        graph = torch.cuda.CUDAGraph()
        out = torch.empty_like(ref)
        side.synchronize()
    with torch.cuda.graph(graph, stream=side):
        binding.dab_pack_activations(X, out=out)
    out.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
