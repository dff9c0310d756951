"""Rows on which the value-bucket search has to take its rarer branches, and sizes at the edges of its kernels: two maxima of D of
nearly the same height (candidate buckets far apart, taken one at a time), buckets of more elements than a cell counts, more
equal values at the split than the list holds, a range far below the largest magnitude, an outlier that leaves one bucket for
all the rest, ties that the index decides, a smallest weight that is rounded away beside the largest.  Every row
against the oracle, through the separate and the grouped calls."""
import numpy as np
import pytest
import torch

from oracle import packing as opk
from paper_1804_02941_amd import binding as dab

import gpu_util as gu
from test_gpu_training import check_bounded

pytestmark = pytest.mark.gpu


def rows(rng, F, n, kind):
    g = rng.standard_normal((F, n))
    if kind == "two_maxima":                                      # heavy tails, symmetric: splits i and n - i score the same
        half = rng.standard_t(2.2, (F, n // 2))
        w = np.concatenate([half, -half, np.zeros((F, n - 2 * (n // 2)))], axis=1)
        w = rng.permuted(w, axis=1)
    elif kind == "pruned":                                        # more than half the row is exactly zero
        w = np.where(rng.random((F, n)) < 0.55, 0.0, g)
    elif kind == "spike":                                         # a third of the row at the value where the split falls
        w = np.where(rng.random((F, n)) < 0.33, 0.01, g)
    elif kind == "far_mean":
        w = 1e-3 * g + np.linspace(0.002, 5.0, F)[:, None]
    elif kind == "outlier":
        w = 0.01 * g
        w[:, n // 3] = 300.0
    elif kind == "grid":                                          # values on a coarse grid: ties everywhere, zeros of both signs
        w = np.round(g * 8) / 8 * np.where(rng.random((F, n)) < 0.5, 1.0, -1.0)
    elif kind == "tiny_minimum":                                  # one weight below 2^-24 of the others, the row's minimum
        w = np.abs(g).astype(np.float32) * np.float32(0.1) + np.float32(0.01)
        k = np.resize([0.6, -0.3, 281.4, 281.6, 282.6, 1e-26], F)
        w[:, n // 3] = np.ldexp(k, np.frexp(w.max(axis=1))[1] - 48)
    else:
        w = g
    return np.ascontiguousarray(w, dtype=np.float32)


KINDS = ["two_maxima", "pruned", "spike", "far_mean", "outlier", "grid", "gauss", "tiny_minimum"]
# chunk edges (four elements of 256 or 512 threads), class limits, rows of a few weights
SIZES = [5, 63, 191, 193, 255, 1023, 1025, 2303, 3071, 3584, 4095, 4608, 4609, 6145, 9215, 9216, 9217, 12544, 13312]


def check_multi(W, shape):
    F = W.shape[0]
    Wt = gu.to_gpu(W.reshape(shape))
    it = dict(W=Wt, est=dab.estimate_outputs(F, Wt.device), packed=dab.pack_weights_outputs(*shape, Wt.device))
    dab.dab_binarize_weights_multi(dab.weight_jobs([it]))
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in it["est"].items()}
    e, _ = gu.check_estimate(W.reshape(shape), got)
    E_ref, ecnt_ref = opk.pack_weights(e)
    assert np.array_equal(gu.u32(it["packed"][0]), E_ref) and np.array_equal(gu.u32(it["packed"][1]), ecnt_ref)


@pytest.mark.parametrize("kind", KINDS)
def test_rows_of_every_size_and_kind(kind):
    rng = np.random.default_rng(KINDS.index(kind) + 50)
    for n in SIZES:
        W = rows(rng, 6, n, kind)
        got, _ = gu.gpu_estimate(W)
        gu.check_estimate(W, got)
        if kind == "tiny_minimum" and n < 63:                     # (a group of the rounded weight alone: its mean is rounded there)
            continue
        check_multi(W, (6, n, 1, 1))
        if n % 9 == 0:
            check_multi(W, (6, n // 9, 3, 3))


@pytest.mark.parametrize("F,n", [(1537, 130), (1537, 2304), (1537, 4100), (513, 9300)])
def test_many_rows(F, n):
    """Enough rows for the forms that launches of many rows take."""
    rng = np.random.default_rng(F + n)
    W = rows(rng, F, n, "gauss")
    W[::7] = rows(rng, len(W[::7]), n, "two_maxima")
    W[5] = 0.5
    got, _ = gu.gpu_estimate(W)
    gu.check_estimate(W, got)
    check_multi(W, (F, n, 1, 1))


@pytest.mark.parametrize("n", [190, 1600, 4096, 9300])
def test_windows_narrower_than_a_bucket(n):
    rng = np.random.default_rng(n)
    W = rows(rng, 24, n, "gauss")
    K_prev = rng.integers(1, n, 24).astype(np.int32)
    upper = rng.integers(0, 2, 24).astype(np.uint8)
    for change in (0, 1, 3, n // 64, n):
        out = dab.dab_estimate_alpha_beta_bounded(gu.to_gpu(W), gu.to_gpu(K_prev), gu.to_gpu(upper), change)
        torch.cuda.synchronize()
        check_bounded(W, {k: v.cpu().numpy() for k, v in out.items()}, K_prev, upper, change)
