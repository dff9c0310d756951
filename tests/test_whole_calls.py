"""Calls of single layers done whole in native code: plain ones return what the binding's Python returns, and everything else is
left to it before anything is launched."""
import os

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_1804_02941_amd import binding as dab
from paper_1804_02941_amd import build

WHOLE = {"pack_activations": 4, "binconv2d": 7, "binconv2d_bits": 8, "binfc": 7, "pool_bits": 7, "wbin_conv2d": 7, "wbin_fc": 6}


@pytest.fixture(scope="module")
def call():
    if not (os.path.exists(dab.LIB_PATH) and os.path.exists(build.CALL)):
        build.build()
    return dab.native()


@pytest.mark.parametrize("name", WHOLE)
def test_what_is_not_plain_is_left_to_python(call, name):
    f, n = getattr(call, name), WHOLE[name]
    with pytest.raises(TypeError, match=f"takes {n} arguments"):
        f(*[None] * (n + 1))
    d = dab.dab_conv_desc(1, 32, 4, 4, 32, 3, 3, 1, 1, 1, 1)
    for x in (None, 3, "x", torch.zeros(2, 64), torch.zeros(2, 64, dtype=torch.int32), torch.zeros(2, 64, device="meta"), d):
        assert f(*[x] * n) is None
        assert f(d, *[x] * (n - 1)) is None


class Mode(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def _calls():
    dev = "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    X = torch.randn(3, 9, 8, 70, generator=g, device=dev)
    tau = torch.randn(70, generator=g, device=dev)
    w = dab.estimate_outputs(50, dev)
    E, cnt = dab.pack_weights_outputs(50, 70, 3, 3, dev)
    dab.dab_binarize_weights_multi(dab.weight_jobs([dict(W=torch.randn(50, 70, 3, 3, generator=g, device=dev), est=w, packed=(E, cnt))]))
    d = dab.dab_conv_desc(3, 70, 9, 8, 50, 3, 3, 1, 1, 2, 2)
    A = dab.dab_pack_activations(X, dab.DAB_LAYOUT_NHWC, tau)
    V = torch.randn(4, 70 * 9, generator=g, device=dev)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=dev)
    Ef, al, be = torch.randint(-2**31, 2**31 - 1, (20, 64), generator=g, device=dev).to(torch.int32), w["alpha"], w["beta"]
    tail = (1 << (630 % 32)) - 1
    Ef[-1] &= tail
    Af = dab.dab_pack_activations(V)
    return {
        "pack_activations": [lambda **k: dab.dab_pack_activations(X, dab.DAB_LAYOUT_NHWC, tau, **k), lambda **k: dab.dab_pack_activations(V, **k),
                             lambda **k: dab.dab_pack_activations(X.permute(0, 3, 1, 2).contiguous(), dab.DAB_LAYOUT_NCHW, **k)],
        "binconv2d": [lambda **k: dab.dab_binconv2d(d, A, E, al, be, **k)],
        "binconv2d_bits": [lambda **k: dab.dab_binconv2d_bits(d, A, E, al, be, None, **k), lambda **k: dab.dab_binconv2d_bits(d, A, E, al, be, al, **k)],
        "binfc": [lambda **k: dab.dab_binfc(Af.view(4, -1), Ef, al, be, 630, **k)],
        "pool_bits": [lambda **k: dab.dab_pool_bits(A, 70, 3, 2, 2, 3, **k)],
        "wbin_conv2d": [lambda **k: dab.dab_wbin_conv2d(d, X, E, al, be, ws=ws, **k)],
        "wbin_fc": [lambda **k: dab.dab_wbin_fc(V, Ef, al, be, ws=ws, **k)],
    }


@pytest.mark.gpu
@pytest.mark.parametrize("name", WHOLE)
def test_plain_calls_return_what_python_returns(call, name, monkeypatch):
    for f in _calls()[name]:
        taken = []
        whole = getattr(call, name)
        proxy = type("Counting", (), {k: staticmethod(getattr(call, k)) for k in dir(call) if not k.startswith("__")})
        setattr(proxy, name, staticmethod(lambda *a: taken.append(whole(*a)) or taken[-1]))
        monkeypatch.setattr(dab, "_native", proxy)
        got = f()
        assert taken[-1] is got                                     # done whole
        out = torch.zeros_like(got)
        assert f(out=out) is out and taken[-1] is out and torch.equal(out, got)
        with Mode():
            moded = f()
        assert taken[-1] is None and torch.equal(moded, got)        # a mode: left to Python
        setattr(proxy, name, staticmethod(lambda *a: None))
        ref = f()
        assert ref.shape == got.shape and ref.dtype == got.dtype and ref.device == got.device and torch.equal(ref, got)
        monkeypatch.setattr(dab, "_native", call)


@pytest.mark.gpu
def test_refusals_are_those_of_the_entry_points(call):
    X = torch.randn(2, 64, device="cuda:0")
    A = dab.dab_pack_activations(X)
    with pytest.raises(TypeError, match="X: expected torch.float32"):
        dab.dab_pack_activations(X.double())
    with pytest.raises(ValueError, match="X: tensor must be contiguous"):
        dab.dab_pack_activations(torch.randn(64, 4, device="cuda:0").t())
    with pytest.raises(dab.DabError, match="dab_binfc failed: status 2"):
        dab.dab_binfc(A.view(2, -1), A, X[0].contiguous(), X[0].contiguous(), 1)
    with pytest.raises(dab.DabError, match="dab_pool_bits failed"):
        dab.dab_pool_bits(A, 64, 3, 3, 1, 1)


@pytest.mark.gpu
@pytest.mark.parametrize("own", [False, True])
def test_calls_that_need_a_workspace_are_done_whole(call, own, monkeypatch):
    """Without a workspace, or with one that is too small, the call makes one itself: one allocation for it and one for the output,
    and what Python returns."""
    dev = "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(6)
    words = lambda *shape: torch.randint(-2**31, 2**31 - 1, shape, generator=g, device=dev).to(torch.int32)
    al, be = torch.rand(1284, generator=g, device=dev), -torch.rand(1284, generator=g, device=dev)
    d = dab.dab_conv_desc(160, 320, 12, 12, 640, 3, 3, 0, 0, 1, 1)
    A, E, Af, Ef = words(160, 12, 12, 10), words(90, 640), words(8192, 75), words(75, 1344)
    Ef[:, 1284:] = 0
    X, V = torch.randn(2, 12, 12, 320, generator=g, device=dev), torch.randn(9, 2400, generator=g, device=dev)
    dw = dab.dab_conv_desc(2, 320, 12, 12, 640, 3, 3, 0, 0, 1, 1)
    assert dab.lib().dab_binconv2d_workspace_bytes(d) > 1 < dab.lib().dab_binfc_workspace_bytes(8192, 2400, 1284)
    ws = torch.empty(1, dtype=torch.uint8, device=dev) if own else None
    for name, f in (("binconv2d", lambda: dab.dab_binconv2d(d, A, E, al, be, ws=ws)),
                    ("binconv2d_bits", lambda: dab.dab_binconv2d_bits(d, A, E, al, be, al, ws=ws)),
                    ("binfc", lambda: dab.dab_binfc(Af, Ef, al, be, 2400, ws=ws)),
                    ("wbin_conv2d", lambda: dab.dab_wbin_conv2d(dw, X, E, al, be, ws=ws)),
                    ("wbin_fc", lambda: dab.dab_wbin_fc(V, Ef, al, be, ws=ws))):
        taken = []
        whole = getattr(call, name)
        proxy = type("Counting", (), {k: staticmethod(getattr(call, k)) for k in dir(call) if not k.startswith("__")})
        setattr(proxy, name, staticmethod(lambda *a: taken.append(whole(*a)) or taken[-1]))
        monkeypatch.setattr(dab, "_native", proxy)
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        got = f()
        assert taken[-1] is got and torch.cuda.memory_stats()["allocation.all.allocated"] - before == 2, name
        setattr(proxy, name, staticmethod(lambda *a: None))
        assert torch.equal(f(), got), name
        monkeypatch.setattr(dab, "_native", call)
