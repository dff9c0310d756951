"""Activation packing, channels last: every way through it, at the ends of words, items and batches."""
import numpy as np
import pytest
import torch

from paper_1804_02941_amd import binding as dab

pytestmark = pytest.mark.gpu

# channels: whole words or not, item counts per pixel that divide a batch of sixteen or do not
CHANNELS = [1, 31, 32, 33, 64, 65, 96, 100, 160, 192, 320, 577, 1024, 1056, 1120, 9216]


def signs(x, tau):
    """x [P, C] -> words [P, ceil(C / 32)]"""
    P, C = x.shape
    bits = np.zeros((P, (C + 31) // 32 * 32), np.uint8)
    bits[:, :C] = x >= (0.0 if tau is None else tau)
    return np.packbits(bits, axis=1, bitorder="little").view(np.uint32)


def inputs(C, pixels):
    rng = np.random.default_rng(C * 7 + pixels)
    x = rng.standard_normal((pixels, C)).astype(np.float32)
    odd = rng.random(x.shape)
    for i, v in enumerate((0.0, -0.0, np.nan, np.inf, -np.inf, np.float32(1e-45), -np.float32(1e-45))):
        x[(odd >= 0.02 * i) & (odd < 0.02 * (i + 1))] = v
    return x, rng.standard_normal(C).astype(np.float32)


@pytest.mark.parametrize("C", CHANNELS)
@pytest.mark.parametrize("pixels", [1, 2, 3, 17, 1031])
def test_each_channel_count(C, pixels):
    x, tau = inputs(C, pixels)
    X = torch.from_numpy(x).to("cuda:0")
    for t in (None, tau):
        T = None if t is None else torch.from_numpy(t).to("cuda:0")
        want = signs(x, t)
        A = dab.dab_pack_activations(X.view(pixels, 1, 1, C), dab.DAB_LAYOUT_NHWC, T)
        assert np.array_equal(A.cpu().numpy().view(np.uint32).reshape(want.shape), want)
        out = torch.full((pixels, 1, 1, want.shape[1]), -1, dtype=torch.int32, device="cuda:0")
        small = torch.full((pixels, 1, 1, want.shape[1]), -1, dtype=torch.int32, device="cuda:0")
        dab.dab_pack_activations_multi(dab.pack_jobs([(X, T, out), (X, T, small)]))
        for a in (out, small):
            assert np.array_equal(a.cpu().numpy().view(np.uint32).reshape(want.shape), want)


def test_more_batches_than_wavefronts():
    """Every wavefront walks over several batches, odd channel counts included."""
    for C, pixels in ((100, 300000), (96, 200000), (2112, 9001)):
        x, tau = inputs(C, pixels)
        X, T = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(tau).to("cuda:0")
        for t, Tt in ((None, None), (tau, T)):
            A = dab.dab_pack_activations(X, dab.DAB_LAYOUT_NHWC, Tt)
            assert np.array_equal(A.cpu().numpy().view(np.uint32).reshape(pixels, -1), signs(x, t))
