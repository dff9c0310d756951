"""The weights-only layer in every form of its two kernels: odd channels, filters and pixels, strides, borders.

Integer inputs small enough that every sum is below 2^24 have to come out exactly, so any wrong index
shows; a lone input has to come out bit for bit, whatever its exponent, because its three pieces are exact.
"""
import numpy as np
import pytest
import torch

from paper_1804_02941_amd import binding as dab

DEV = "cuda:0"

# (kernel, (rows or 0, filter blocks, wavefronts along the pixels or shares of the reduction)) -> B, C, H, W, F, k, pad, stride
FORMS = {
    (0, 4, 4): [(7, 70, 41, 38, 130, 3, 1, 1), (128, 48, 10, 23, 150, 2, 0, 1)],
    (0, 2, 4): [(40, 70, 36, 18, 1, 2, 1, 1), (40, 48, 53, 12, 1, 2, 1, 1), (128, 17, 22, 16, 1, 5, 0, 1)],
    (0, 2, 2): [(128, 70, 15, 50, 65, 3, 0, 2), (19, 17, 22, 42, 33, 5, 2, 1)],
    (32, 4, 1): [(19, 40, 58, 32, 65, 1, 0, 1), (19, 48, 45, 42, 65, 2, 1, 1)],
    (32, 2, 1): [(40, 70, 33, 35, 1, 2, 1, 1), (40, 40, 27, 16, 1, 1, 0, 1)],
    (32, 4, 4): [(7, 70, 39, 32, 65, 2, 1, 1), (7, 17, 59, 59, 130, 5, 2, 2)],
    (32, 2, 4): [(40, 70, 4, 43, 1, 2, 1, 1), (3, 17, 57, 51, 33, 5, 2, 1)],
    (32, 2, 8): [(7, 70, 39, 59, 33, 2, 1, 2), (2, 17, 37, 60, 33, 5, 2, 1)],
    (32, 1, 8): [(19, 70, 8, 25, 1, 2, 1, 1), (128, 17, 34, 1, 1, 5, 2, 1), (40, 40, 35, 12, 1, 1, 0, 2)],
    (16, 4, 8): [(300, 1000, 1, 1, 520, 1, 0, 1), (7, 17, 6, 49, 33, 5, 2, 1)],
    (16, 2, 8): [(2, 70, 54, 12, 33, 2, 1, 1), (1, 17, 41, 25, 50, 5, 2, 1)],
    (16, 1, 8): [(1, 70, 35, 3, 1, 3, 0, 2), (1, 3, 2, 4, 1, 3, 1, 2), (3, 333, 1, 1, 30, 1, 0, 1)],
}
LAYERS = [(form, layer) for form, layers in FORMS.items() for layer in layers]


def run(layer, x, e, alpha, beta):
    """x [B,H,W,C] and the mask e [F,C,k,k] through the packing and the layer call."""
    B, C, H, W, F, k, pad, stride = layer
    half = torch.full((F,), 0.5, device=DEV)
    zeros = torch.zeros(F, dtype=torch.int32, device=DEV)
    E, _ = dab.dab_pack_weights(e.to(DEV), half, zeros, torch.ones(F, dtype=torch.uint8, device=DEV))
    a, b = (torch.full((F,), v, device=DEV) for v in (alpha, beta))
    if H == W == k == 1:
        return dab.dab_wbin_fc(x.view(B, C), E, a, b).view(B, 1, 1, F)
    return dab.dab_wbin_conv2d(dab.dab_conv_desc(B, C, H, W, F, k, k, pad, pad, stride, stride), x, E, a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("form,layer", LAYERS, ids=["%s-%s" % ("_".join(map(str, f)), "x".join(map(str, l))) for f, l in LAYERS])
def test_integer_inputs_are_exact(form, layer):
    B, C, H, W, F, k, pad, stride = layer
    rng = torch.Generator().manual_seed(C * 1000 + F)
    peak = min(2 ** 12, 2 ** 24 // (3 * C * k * k) - 1)              # |3 x| summed over the window stays below 2^24
    x = torch.randint(-peak, peak + 1, (B, H, W, C), generator=rng).float()
    e = torch.randint(0, 2, (F, C, k, k), generator=rng).float()
    Y = run(layer, x.to(DEV), e, 3.0, 1.0)                            # 2 s1 + the window sum
    ref = torch.nn.functional.conv2d(x.permute(0, 3, 1, 2).double(), 2.0 * e.double() + 1.0, padding=pad, stride=stride)
    assert torch.equal(Y.cpu().double(), ref.permute(0, 2, 3, 1))


@pytest.mark.gpu
@pytest.mark.parametrize("layer", [(64, 100, 1, 1, 40, 1, 0, 1), (2000, 70, 1, 1, 130, 1, 0, 1), (40, 20, 13, 32, 65, 3, 1, 1)])
def test_a_lone_input_comes_out_bit_for_bit(layer):
    B, C, H, W, F, k, pad, stride = layer
    rng = np.random.default_rng(5)
    x = np.zeros((B, H, W, C), np.float32)
    # one nonzero value an image, in its middle; every mantissa, exponents whose last piece is a normal number
    v = (rng.integers(0, 2, B) << 31 | rng.integers(30, 250, B) << 23 | rng.integers(0, 1 << 23, B)).astype(np.uint32).view(np.float32)
    c = rng.integers(0, C, B)
    x[np.arange(B), H // 2, W // 2, c] = v
    e = (rng.random((F, C, k, k)) < 0.5).astype(np.float32)
    Y = run(layer, torch.from_numpy(x).to(DEV), torch.from_numpy(e), 1.0, 0.0).cpu().numpy()
    want = np.zeros_like(Y)
    for i in range(B):
        for ky in range(k):
            for kx in range(k):
                oy, ox = H // 2 + pad - ky, W // 2 + pad - kx
                want[i, oy, ox] = e[:, c[i], ky, kx] * v[i]
    assert np.array_equal(Y, want)
