"""The kernels that hold a filter in registers, at the edges of their classes: centring, W~, the gradient factor and the packed
mask of rows one weight short of, at and past every class limit, as whole 16-byte pieces and not, from pointers that are
16-byte aligned and not, out of place and in place; filters at the limits of the packing kernels' rows and taps."""
import numpy as np
import pytest
import torch

from oracle import packing as opk
from oracle import training as otr
from paper_1804_02941_amd import binding as dab

import gpu_util as gu

pytestmark = pytest.mark.gpu

RTOL = 1e-6                                                       # one fp32 rounding of a float64 value, as in test_gpu_training.py
LIMITS = [512, 1024, 2048, 4096, 8192, 14336, 16384]
ROWS = sorted({2, 3, 4, 7, 300} | {L + d for L in LIMITS for d in (-1, 0, 1, 4)} | {40001})


def at_offset(a, off):
    """a on the GPU, its first element `off` floats behind a 16-byte boundary."""
    t = torch.empty(a.size + 4, dtype=torch.float32, device=gu.DEV)
    v = t[off:off + a.size].view(a.shape)
    v.copy_(gu.to_gpu(a))
    return v


@pytest.mark.parametrize("off", [0, 1])
def test_training_rows_at_class_edges(off):
    rng = np.random.default_rng(11 + off)
    for n in ROWS:
        F = 3
        W = (0.7 * rng.standard_normal((F, n))).astype(np.float32)
        up = rng.standard_normal((F, n)).astype(np.float32)
        ti = rng.integers(0, n, F)
        tv = W[np.arange(F), ti].copy()
        W[1, ::5] = tv[1]                                         # ties that the index decides
        upper = np.array([1, 0, 1], np.uint8)
        lower = (W < tv[:, None]) | ((W == tv[:, None]) & (np.arange(n)[None] <= ti[:, None]))
        e = (lower != upper[:, None].astype(bool)).astype(np.uint8)
        if not (np.all(e.sum(1) > 0) and np.all(e.sum(1) < n)):  # a group without members is outside the theorem
            continue
        d = [gu.to_gpu(tv), gu.to_gpu(ti.astype(np.int32)), gu.to_gpu(upper)]
        al, be = gu.to_gpu(np.float32([2, 3, 4])), gu.to_gpu(np.float32([-5, -6, -7]))
        x, u = at_offset(W, off), at_offset(up, off)
        got = [dab.dab_mean_center_clamp(x.view(F, n, 1, 1)).view(F, n), dab.dab_binarized_weights(x, al, be, *d),
               dab.dab_weight_gradient(x, *d), dab.dab_weight_gradient(x, *d, upstream=u)]
        want = [otr.mean_center_clamp(W.reshape(F, n, 1, 1)).reshape(F, n),
                np.where(e == 1, al.cpu().numpy()[:, None], be.cpu().numpy()[:, None]), otr.weight_gradient(W, e),
                otr.weight_gradient(W, e, up)]
        for k, (g, w) in enumerate(zip(got, want)):
            assert np.allclose(g.cpu().numpy(), w, rtol=RTOL, atol=1e-7 if k == 0 else 0), (n, k)
        # in place: the same bits
        for k, f in enumerate((lambda t: dab.dab_mean_center_clamp(t.view(F, n, 1, 1), out=t.view(F, n, 1, 1)),
                               lambda t: dab.dab_binarized_weights(t, al, be, *d, out=t),
                               lambda t: dab.dab_weight_gradient(t, *d, out=t),
                               lambda t: dab.dab_weight_gradient(t, *d, upstream=u, out=t))):
            t = at_offset(W, off)
            f(t)
            assert torch.equal(t, got[k]), (n, k)


# (C, kh, kw): one tap and windows around the classes' rows (1024, 2304, 4608, 9216, 13312), the row past them, as many taps as
# the row kernels count and one more, channel counts that end inside a word
FILTERS = [(2, 1, 1), (31, 1, 1), (1024, 1, 1), (1025, 1, 1), (2304, 1, 1), (2305, 1, 1), (4608, 1, 1), (4609, 1, 1), (9217, 1, 1),
           (13312, 1, 1), (13313, 1, 1), (114, 3, 3), (256, 3, 3), (257, 3, 3), (100, 8, 16), (70, 129, 1), (271, 7, 7), (272, 7, 7),
           (33, 5, 5), (1024, 3, 3)]


@pytest.mark.parametrize("F", [3, 65])
def test_packed_masks_at_class_edges(F):
    rng = np.random.default_rng(F)
    for C, kh, kw in FILTERS:
        n = C * kh * kw
        W = np.round(rng.standard_normal((F, n)) * 16).astype(np.float32) / 16          # many ties, zeros among them
        W[:, ::7] *= -1                                                                 # (both zeros)
        ti = rng.integers(0, n, F).astype(np.int32)
        tv = W[np.arange(F), ti].copy()
        tv[0], ti[0] = -np.inf, 0                                                       # nothing is lower
        upper = rng.integers(0, 2, F).astype(np.uint8)
        upper[0] = 1
        lower = (W < tv[:, None]) | ((W == tv[:, None]) & (np.arange(n)[None] <= ti[:, None]))
        e = (lower != upper[:, None].astype(bool)).astype(np.uint8).reshape(F, C, kh, kw)
        E, ecnt = dab.pack_weights_outputs(F, C, kh, kw, gu.DEV)
        E.fill_(-1)
        ecnt.fill_(-1)
        dab.dab_pack_weights(gu.to_gpu(W.reshape(F, C, kh, kw)), gu.to_gpu(tv), gu.to_gpu(ti), gu.to_gpu(upper), out=(E, ecnt))
        E_ref, ecnt_ref = opk.pack_weights(e)
        assert np.array_equal(gu.u32(E), E_ref) and np.array_equal(gu.u32(ecnt), ecnt_ref), (C, kh, kw)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_the_gradient_of_a_group_does_not_see_the_other_groups_infinity(bad):
    rng = np.random.default_rng(5)
    for n in (300, 1024, 4097, 16384, 20000):
        W = (0.7 * rng.standard_normal((2, n))).astype(np.float32)
        W[:, n // 2] = bad
        upper = np.array([1, 0], np.uint8)                        # the alpha group, then the other one, holds +inf and NaN
        lower = W < 0.25
        d = [gu.to_gpu(np.full(2, 0.25, np.float32)), gu.to_gpu(np.full(2, -1, np.int32)), gu.to_gpu(upper)]
        got = dab.dab_weight_gradient(gu.to_gpu(W), *d).cpu().numpy()
        for f in range(2):
            rest = lower[f] if bad != -np.inf else ~lower[f]      # the group without it
            w = W[f][rest].astype(np.float64)
            ref = 1 / rest.sum() + np.abs(w).sum() / rest.sum() * np.where(np.abs(w) <= 1, w, 0)
            assert np.allclose(got[f][rest], ref, rtol=RTOL, atol=0), (n, f)
