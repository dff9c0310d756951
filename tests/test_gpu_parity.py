"""GPU parity tests: every C-ABI entry point against the CPU oracle, element by element.

Integers (packed bits, per-tap counts, K, s1) must match exactly; alpha/beta to 1e-6
relative; the fp32 layer output to 1e-5 relative (see gpu_util.Y_RTOL).  Sizes are small
enough for the oracle to finish in seconds but span several workgroup tiles and ragged
tails.  Full-size runs are in test_gpu_fullsize.py.
"""
import numpy as np
import pytest
import torch

from oracle import estimate as oest
from oracle import layers as olay
from oracle import packing as opk
from paper_1804_02941_amd import binding as dab
from paper_1804_02941_amd import workloads as wl
from paper_1804_02941_amd.workloads import Layer

import gpu_util as gu

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------ dab_pack_activations
@pytest.mark.parametrize("C", [1, 31, 32, 33, 64, 65, 96, 100, 128, 256, 512])
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
def test_pack_activations(C, layout):
    rng = np.random.default_rng(C)
    B, H, W = 3, 5, 7
    x = rng.standard_normal((B, C, H, W)).astype(np.float32)
    x[0, 0, 0, 0] = 0.0
    x[0, C - 1, 0, 1] = -0.0
    x[1, 0, 1, 1] = np.nan
    x[2, C // 2, 2, 2] = np.inf
    for tau in (None, rng.standard_normal(C).astype(np.float32) * 0.5):
        ref = opk.pack_activations(olay.binarize_activations(x, tau))
        tt = gu.to_gpu(tau) if tau is not None else None
        if layout == "nhwc":
            A = dab.dab_pack_activations(gu.to_gpu(np.transpose(x, (0, 2, 3, 1))), dab.DAB_LAYOUT_NHWC, tt)
        else:
            A = dab.dab_pack_activations(gu.to_gpu(x), dab.DAB_LAYOUT_NCHW, tt)
        torch.cuda.synchronize()
        assert np.array_equal(gu.u32(A), ref)


def test_pack_activations_fc_and_ragged_sizes():
    rng = np.random.default_rng(5)
    for B, C in ((1, 2), (7, 9216), (130, 4096), (1025, 70), (3, 12544)):
        x = rng.standard_normal((B, C)).astype(np.float32)
        ref = opk.pack_activations(olay.binarize_activations(x))
        A = dab.dab_pack_activations(gu.to_gpu(x))
        torch.cuda.synchronize()
        assert np.array_equal(gu.u32(A).reshape(ref.shape), ref)


def test_pack_activations_multi():
    """Several tensors in one launch: bit for bit the oracle's packing of each (and so the separate calls')."""
    rng = np.random.default_rng(99)
    shapes = [(3, 5, 7, 64), (2, 9, 4, 128), (5, 3, 3, 256), (1, 2, 2, 512), (4, 6, 5, 1024), (7, 1, 1, 70), (130, 1, 1, 4096),
              (2, 4, 4, 1), (3, 2, 5, 96), (1, 1, 1, 2048)]
    items, refs = [], []
    for k, (B, H, W, C) in enumerate(shapes):
        x = rng.standard_normal((B, C, H, W)).astype(np.float32)
        tau = None if k % 3 == 0 else (rng.standard_normal(C) * 0.5).astype(np.float32)
        refs.append(opk.pack_activations(olay.binarize_activations(x, tau)))
        X = gu.to_gpu(np.transpose(x, (0, 2, 3, 1)))
        items.append((X, gu.to_gpu(tau) if tau is not None else None,
                      torch.full((B, H, W, dab.words_per_pixel(C)), -1, dtype=torch.int32, device=gu.DEV)))
    dab.dab_pack_activations_multi(dab.pack_jobs(items))
    torch.cuda.synchronize()
    for (X, tau, A), ref in zip(items, refs):
        assert np.array_equal(gu.u32(A), ref)
    # a single job, and too many jobs
    dab.dab_pack_activations_multi(dab.pack_jobs(items[:1]))
    with pytest.raises(dab.DabError) as ei:
        dab.dab_pack_activations_multi(dab.pack_jobs(items * 2))
    assert ei.value.status == 5
    torch.cuda.synchronize()


# ------------------------------------------------------------------ dab_estimate_alpha_beta
def weight_rows(rng, F, n, kind):
    if kind == "gauss":
        return (rng.standard_normal((F, n)) * 0.05 + rng.uniform(-0.02, 0.02, (F, 1))).astype(np.float32)
    if kind == "laplace":
        return rng.laplace(0.004, 0.03, (F, n)).astype(np.float32)
    if kind == "mixture":
        return wl.skewed_mixture_weights(rng, rng, F, n, n)
    if kind == "dupes":
        return (np.round(rng.standard_normal((F, n)) * 6) / 16).astype(np.float32)
    if kind == "onesided":
        return np.abs(rng.standard_normal((F, n))).astype(np.float32) + 0.25
    raise ValueError(kind)


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 256, 257, 576, 768, 769, 1024, 1025, 1600, 2304, 2817, 3072, 3073, 3585, 4095, 4096,
                               4608, 5120, 5121, 8192, 8193, 9216, 12544, 13312])
def test_estimate_sizes(n):
    rng = np.random.default_rng(n)
    F = 6 if n > 3000 else 10
    W = np.concatenate([weight_rows(rng, F // 2, n, "gauss"), weight_rows(rng, F - F // 2, n, "mixture")])
    got, _ = gu.gpu_estimate(W)
    _, differ = gu.check_estimate(W, got)
    assert differ <= 1


@pytest.mark.parametrize("n", [150, 700, 1200, 1600, 1792, 2304, 2816, 3000, 3584, 4608, 5632, 7168, 9216, 11264, 13312])
def test_estimate_many_filters_share_compute_units(n):
    """Every kernel configuration with several workgroups resident per compute unit.

    1536 filters in one launch put up to six workgroups on a compute unit; the same rows estimated
    128 at a time (at most one workgroup per unit) must give identical results, and a sample of
    the rows is checked against the oracle.  Regression test: configurations whose register
    allocation was exactly 64 VGPRs passed alone and failed as soon as workgroups shared a unit.
    """
    rng = np.random.default_rng(1000 + n)
    F = 1536
    W = (rng.standard_normal((F, n)) * 0.05).astype(np.float32)
    Wt = gu.to_gpu(W)
    whole = dab.dab_estimate_alpha_beta(Wt)
    again = dab.dab_estimate_alpha_beta(Wt)
    parts = [dab.dab_estimate_alpha_beta(Wt[f0:f0 + 128].contiguous()) for f0 in range(0, F, 128)]
    torch.cuda.synchronize()
    for key in whole:
        chunks = torch.cat([p[key] for p in parts])
        assert torch.equal(whole[key], chunks), f"{key}: one launch differs from 128-filter launches"
        assert torch.equal(whole[key], again[key]), f"{key}: two identical launches differ"
    pick = rng.choice(F, size=24, replace=False)
    got = {k: v.cpu().numpy()[pick] for k, v in whole.items()}
    gu.check_estimate(W[pick], got)


@pytest.mark.parametrize("kind", ["gauss", "laplace", "mixture", "dupes", "onesided"])
def test_estimate_distributions(kind):
    rng = np.random.default_rng(17)
    W = weight_rows(rng, 40, 777, kind)
    got, _ = gu.gpu_estimate(W)
    gu.check_estimate(W, got)


def test_estimate_degenerate_rows():
    n = 200
    rows = [
        np.full(n, 0.25, np.float32),                                         # constant
        np.concatenate([np.zeros(n // 2), -np.zeros(n // 2)]).astype(np.float32),   # +0 / -0 only
        np.concatenate([np.full(n - 1, -1.0), [3.0]]).astype(np.float32),     # one outlier
        np.concatenate([np.full(n // 2, -0.5), np.full(n // 2, 0.5)]).astype(np.float32),   # symmetric two-point
        np.arange(n, dtype=np.float32) / n,                                   # already sorted
        -np.arange(n, dtype=np.float32) / n,                                  # reverse sorted
    ]
    W = np.stack(rows)
    got, _ = gu.gpu_estimate(W)
    e, differ = gu.check_estimate(W, got)
    assert differ == 0
    assert got["K"][0] == 1 and got["thr_idx"][0] == n - 2
    assert got["K"][3] == n // 2 and got["alpha"][3] == 0.5 and got["beta"][3] == -0.5


@pytest.mark.parametrize("kind", ["gauss", "laplace", "mixture", "dupes", "onesided"])
@pytest.mark.parametrize("n", [4096, 5003, 12544])
def test_estimate_long_rows(kind, n):
    """Rows long enough for the bucket kernel (value buckets, bounds, exact ranking of the few
    candidates), including rows it hands over to the sort kernel (many equal values)."""
    rng = np.random.default_rng(n + len(kind))
    W = weight_rows(rng, 7, n, kind)
    got, _ = gu.gpu_estimate(W)
    _, differ = gu.check_estimate(W, got)
    assert differ <= 1


@pytest.mark.parametrize("n", [600, 1500, 3700, 6000])
def test_estimate_long_degenerate_rows(n):
    """Rows the value buckets cannot finish (handed to the sort, inside the kernel for short rows and
    in a second launch for long ones) and rows that stress the bucket range and the fixed-point sums."""
    rng = np.random.default_rng(61)
    wide = (rng.standard_normal(n) * np.exp(rng.uniform(-30, 0, n))).astype(np.float32)     # 13 decades of magnitudes
    tiny = (rng.standard_normal(n) * 1e-41).astype(np.float32)                             # denormals only
    outl = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    outl[17] = 250.0                                                                       # one huge value: the rest shares few buckets
    two = np.where(rng.random(n) < 0.3, 0.25, -0.125).astype(np.float32)
    near = (1.0 + rng.integers(0, 50, n) * 2.0 ** -23).astype(np.float32)                  # 50 neighbouring floats
    rows = [
        np.full(n, 0.25, np.float32),                                         # constant
        np.concatenate([np.zeros(n // 2), -np.zeros(n // 2)]).astype(np.float32),   # +0 / -0 only
        np.concatenate([np.full(n - 1, -1.0), [3.0]]).astype(np.float32),     # one outlier among equal values
        two, np.arange(n, dtype=np.float32) / n, -np.arange(n, dtype=np.float32) / n,
        wide, tiny, outl, near,
    ]
    W = np.stack(rows)
    got, _ = gu.gpu_estimate(W)
    _, differ = gu.check_estimate(W, got)
    assert differ <= 1
    assert got["K"][0] == 1 and got["thr_idx"][0] == n - 2
    # the same rows without a workspace (sort kernel only) give the same splits
    t = gu.to_gpu(W)
    out = dab.estimate_outputs(W.shape[0], t.device)
    rc = dab.lib().dab_estimate_alpha_beta(t.data_ptr(), W.shape[0], n, out["alpha"].data_ptr(), out["beta"].data_ptr(),
                                           out["K"].data_ptr(), out["thr_val"].data_ptr(), out["thr_idx"].data_ptr(),
                                           out["alpha_is_upper"].data_ptr(), None, 0, None)
    torch.cuda.synchronize()
    assert rc == 0
    plain = {k: v.cpu().numpy() for k, v in out.items()}
    gu.check_estimate(W, plain)


def test_estimate_xnor_special_case():
    """Symmetric filter: K = n/2 and alpha = -beta = mean|W| (Section 4.2's XNOR-Net simulation)."""
    rng = np.random.default_rng(23)
    h = np.abs(rng.standard_normal((8, 300))).astype(np.float32) + 0.01
    W = np.concatenate([h, -h], axis=1)
    W = np.take_along_axis(W, rng.permuted(np.tile(np.arange(600), (8, 1)), axis=1), axis=1)
    got, _ = gu.gpu_estimate(W)
    assert np.all(got["K"] == 300) and np.all(got["alpha_is_upper"] == 1)
    assert np.allclose(got["alpha"], np.abs(W.astype(np.float64)).mean(axis=1), rtol=1e-6)
    assert np.allclose(got["alpha"], -got["beta"], rtol=1e-6)


# ------------------------------------------------------------------ dab_pack_weights
@pytest.mark.parametrize("F,C,kh,kw", [(5, 3, 1, 1), (64, 64, 3, 3), (70, 45, 2, 3), (130, 100, 5, 5),
                                       (9, 256, 7, 7), (33, 9216, 1, 1), (3, 13000, 1, 1), (4, 330, 3, 3),
                                       (2, 700, 7, 7), (3, 30000, 1, 1)])    # the last two: filters longer than one LDS slab
def test_pack_weights_with_oracle_split(F, C, kh, kw):
    """The packer alone, fed the oracle's split descriptor: bits and counts exact."""
    rng = np.random.default_rng(F * C)
    n = C * kh * kw
    W = weight_rows(rng, F, n, "dupes" if C == 45 else "laplace").reshape(F, C, kh, kw)
    r = oest.estimate_alpha_beta(W)
    E, ecnt = dab.dab_pack_weights(gu.to_gpu(W), gu.to_gpu(r["thr_val"].astype(np.float32)),
                                   gu.to_gpu(r["thr_idx"].astype(np.int32)), gu.to_gpu(r["alpha_is_upper"].astype(np.uint8)))
    torch.cuda.synchronize()
    E_ref, ecnt_ref = opk.pack_weights(r["e"])
    assert np.array_equal(gu.u32(E), E_ref)
    assert np.array_equal(gu.u32(ecnt), ecnt_ref)
    assert np.array_equal(gu.u32(ecnt).sum(axis=1), r["K"])


# ------------------------------------------------------------------ layers, end to end
SMALL_LAYERS = [
    Layer("c3x3_pad", C=37, H=6, W=5, F=7, kh=3, kw=3, pad=1),
    Layer("c3x5_stride", C=100, H=11, W=10, F=70, kh=3, kw=3, pad=1, stride=2),
    Layer("c5x5_pad2_s2", C=33, H=9, W=9, F=5, kh=5, kw=5, pad=2, stride=2),
    Layer("whole_image", C=70, H=7, W=7, F=130, kh=7, kw=7),
    Layer("pointwise", C=3, H=4, W=4, F=3, kh=1, kw=1),
    Layer("c64", C=64, H=12, W=13, F=64, kh=3, kw=3, pad=1),
    Layer("c96_f100", C=96, H=9, W=8, F=100, kh=3, kw=3),
    Layer("wide", C=32, H=3, W=40, F=16, kh=3, kw=3, pad=1),
    # pixels of eight and sixteen words (the small-product kernel's 16-byte activation loads), with padding
    Layer("c256_pad", C=256, H=5, W=6, F=40, kh=3, kw=3, pad=1),
    Layer("c512_pad_s2", C=512, H=7, W=7, F=33, kh=3, kw=3, pad=1, stride=2),
]


@pytest.mark.parametrize("pad", [0, 7])
def test_large_kernel_extent(pad):
    """A 15 x 15 kernel (225 taps, the extent of Sketch-A-Net's first layer), with and without padding."""
    L = Layer(f"k15_pad{pad}", C=6, H=33, W=31, F=20, kh=15, kw=15, pad=pad, stride=3)
    rng = np.random.default_rng(1500 + pad)
    x = rng.standard_normal((2, L.C, L.H, L.W)).astype(np.float32)
    gu.check_layer(L, x, weight_rows(rng, L.F, L.n, "mixture"), tau=None, layout="nhwc")


@pytest.mark.parametrize("L", SMALL_LAYERS, ids=lambda L: L.name)
@pytest.mark.parametrize("B", [1, 3])
def test_small_conv_layers(L, B):
    import zlib
    rng = np.random.default_rng(zlib.crc32(L.name.encode()) % 1000 + B)    # (hash() of a string is salted per process)
    x = rng.standard_normal((B, L.C, L.H, L.W)).astype(np.float32)
    W = weight_rows(rng, L.F, L.n, "mixture")
    gu.check_layer(L, x, W, tau=None, layout="nhwc")
    gu.check_layer(L, x, W, tau=(rng.standard_normal(L.C) * 0.3).astype(np.float32), layout="nchw")


# Layers with enough output pixels for the one-launch kernel that reads both operands as bits
# (at least 129 tiles of 256 pixels), one per load width / padding / odd-word-count variant, with
# ragged pixel and filter tails; the filter counts stay small so that the oracle finishes in seconds.
MANY_PIXEL_LAYERS = [
    (90, Layer("m_c37_pad", C=37, H=20, W=21, F=7, kh=3, kw=3, pad=1)),            # one word per load
    (340, Layer("m_c70_odd", C=70, H=12, W=12, F=130, kh=3, kw=3)),                 # three words per pixel, F % 4 != 0
    (345, Layer("m_c128", C=128, H=10, W=10, F=36, kh=3, kw=3, pad=1)),             # two words per load
    (421, Layer("m_c256", C=256, H=9, W=9, F=20, kh=3, kw=3, pad=1)),               # four words per load
    (341, Layer("m_c33_5x5_s2", C=33, H=19, W=19, F=5, kh=5, kw=5, pad=2, stride=2)),
    (350, Layer("m_c64_5x5", C=64, H=14, W=14, F=12, kh=5, kw=5)),                  # 25 groups: queue depth five
    (1100, Layer("m_pointwise", C=3, H=6, W=6, F=3, kh=1, kw=1)),
    (140, Layer("m_c96_rect", C=96, H=18, W=17, F=64, kh=2, kw=3, pad=1)),
]


@pytest.mark.parametrize("B,L", MANY_PIXEL_LAYERS, ids=lambda v: v.name if isinstance(v, Layer) else str(v))
def test_layers_with_many_pixels(B, L):
    import zlib
    rng = np.random.default_rng(zlib.crc32(L.name.encode()))
    assert dab.lib().dab_binconv2d_workspace_bytes(
        dab.dab_conv_desc(B, L.C, L.H, L.W, L.F, L.kh, L.kw, L.pad, L.pad, L.stride, L.stride)) == 0   # the one-launch kernel
    x = rng.standard_normal((B, L.C, L.H, L.W)).astype(np.float32)
    W = weight_rows(rng, L.F, L.n, "mixture")
    tau = (rng.standard_normal(L.C) * 0.3).astype(np.float32)
    gu.check_layer(L, x, W, tau=tau)
    # the re-binarizing epilogue of the same kernel: identical to packing its fp32 output
    g = gu.gpu_layer(L, x, W, tau, want_s1=False)
    est = {k: gu.to_gpu(v) for k, v in g["est"].items()}
    d = dab.dab_conv_desc(B, L.C, L.H, L.W, L.F, L.kh, L.kw, L.pad, L.pad, L.stride, L.stride)
    tau_out = gu.to_gpu((rng.standard_normal(L.F) * np.abs(g["Y"]).mean()).astype(np.float32))
    bits = dab.dab_binconv2d_bits(d, gu.to_gpu(g["A"].view(np.int32)), gu.to_gpu(g["E"].view(np.int32)), est["alpha"],
                                  est["beta"], tau_out)
    ref = dab.dab_pack_activations(g["Y_gpu"], dab.DAB_LAYOUT_NHWC, tau_out)
    torch.cuda.synchronize()
    assert torch.equal(bits, ref)


def test_fc_with_many_rows():
    rng = np.random.default_rng(4242)
    B, K, F = 40000, 200, 9                                    # seven words per row (odd), 157 tiles
    L = Layer("fc_rows", C=K, H=1, W=1, F=F, kh=1, kw=1)
    assert dab.lib().dab_binfc_workspace_bytes(B, K, F) == 0
    x = rng.standard_normal((B, K)).astype(np.float32)
    gu.check_layer(L, x, weight_rows(rng, F, K, "gauss"))


@pytest.mark.parametrize("B,K,F", [(1, 2, 1), (5, 70, 9), (64, 512, 512), (65, 1000, 130), (70, 1280, 96), (300, 4096, 48), (130, 9216, 40)])
def test_small_fc_layers(B, K, F):
    rng = np.random.default_rng(B + K + F)
    L = Layer("fc", C=K, H=1, W=1, F=F, kh=1, kw=1)
    x = rng.standard_normal((B, K)).astype(np.float32)
    W = weight_rows(rng, F, K, "gauss" if K > 2 else "onesided")
    gu.check_layer(L, x, W)


def test_config1_tiny_layer():
    L, x, w = wl.config1()
    gu.check_layer(L, x, w)                                  # half-normal input: every bit is 1
    gu.check_layer(L, x, w, tau=x.mean(axis=(0, 2, 3)))      # mixed bits


def test_config2_shape_small_batch():
    L, x, w = wl.config2(batch=3)
    gu.check_layer(L, x, w, tau=x.mean(axis=(0, 2, 3)))


def test_all_plus_one_input_gives_filter_sums():
    """Non-negative input with tau = 0: every bit is 1 and a valid conv returns sum_i w~_i = sum_i w_i."""
    L, x, w = wl.config2(batch=2)
    g = gu.gpu_layer(L, x, w)
    T = w.astype(np.float64).reshape(L.F, -1).sum(axis=1)
    scale = np.abs(w.astype(np.float64)).reshape(L.F, -1).sum(axis=1)
    assert np.all(np.abs(g["Y"] - T) <= 2e-6 * scale)
    assert np.array_equal(g["s1"], np.broadcast_to(g["est"]["K"], g["s1"].shape))


def test_config3_layers_small_batch():
    """Sketch-A-Net trunk, batch 2, chained through the oracle; each layer checked on identical inputs."""
    B = 2
    imgs = wl.sketch_images(B)
    w1, ws = wl.config3_weights()
    x = wl.config3_conv1_features(imgs, w1).numpy()
    for L, W in zip(wl.CFG3_LAYERS, ws):
        if L.is_fc:
            x = x.reshape(B, -1)
        tau = x.mean(axis=(0, 2, 3)) if x.ndim == 4 else x.mean(axis=0)
        gu.check_layer(L, x, W, tau=tau.astype(np.float32))
        # the next layer's input: this layer's oracle output (float64 -> fp32), pooled where the net pools
        r = oest.estimate_alpha_beta(W)
        a = olay.binarize_activations(x if x.ndim == 4 else x[:, :, None, None], tau.astype(np.float32))
        y = olay.conv2d(a, olay.two_valued_filters(r["e"], r["alpha"], r["beta"]), (L.pad, L.pad), (L.stride, L.stride))
        y = torch.from_numpy(y.astype(np.float32)).permute(0, 3, 1, 2)
        if L.pool_after:
            y = torch.nn.functional.max_pool2d(y, 3, 2)
        x = y.numpy()


@pytest.mark.parametrize("stage", [0, 1, 2, 3])
def test_config4_stages_small_batch(stage):
    L, x, w = wl.config4(stage, batch=1 if stage == 0 else 2)
    gu.check_layer(L, x, w)


@pytest.mark.parametrize("which", [0, 1])
def test_config5_reduced(which):
    L, x, w = wl.config5(which, batch=96, filters=72)
    gu.check_layer(L, x, w)


# ------------------------------------------------------------------ error paths (host validation only)
def test_error_codes():
    lib = dab.lib()
    x = torch.zeros(64, device=gu.DEV)
    a = torch.zeros(64, dtype=torch.int32, device=gu.DEV)
    assert lib.dab_pack_activations(None, 0, 1, 1, 1, 1, None, a.data_ptr(), None) == 1
    assert lib.dab_pack_activations(x.data_ptr(), 0, 0, 1, 1, 1, None, a.data_ptr(), None) == 2
    assert lib.dab_pack_activations(x.data_ptr(), 7, 1, 1, 1, 1, None, a.data_ptr(), None) == 2
    assert lib.dab_pack_activations(x.data_ptr(), 0, 1, 1, 1, 1, None, a.data_ptr() + 4, None) == 3
    with pytest.raises(dab.DabError):
        dab.dab_estimate_alpha_beta(torch.zeros((3, 1), device=gu.DEV))
    with pytest.raises(dab.DabError) as ei:
        dab.dab_estimate_alpha_beta(torch.zeros((1, lib.dab_estimate_max_n() + 1), device=gu.DEV))
    assert ei.value.status == 5
    with pytest.raises(TypeError):
        dab.dab_pack_activations(torch.zeros((1, 4)))        # CPU tensor: no fallback
    torch.cuda.synchronize()


# ------------------------------------------------------------------ the sign-split baseline (XNOR-Net / BWN)
@pytest.mark.parametrize("n", [1, 2, 63, 600, 1600, 20000])
def test_sign_split_estimate_and_layer(n):
    rng = np.random.default_rng(n)
    F = 37
    W = weight_rows(rng, F, n, "dupes" if n == 600 else "gauss")
    if n >= 63:
        W[0] = np.abs(W[0]) + 0.5          # no negative weight
        W[1] = -np.abs(W[1]) - 0.5         # no non-negative weight
        W[2, ::3] = 0.0
        W[2, 1::3] = -0.0
    out = dab.dab_estimate_sign_split(gu.to_gpu(W))
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    ref = oest.estimate_sign_split(W)
    assert np.array_equal(got["K"], ref["K"])
    assert np.array_equal(got["thr_val"].astype(np.float64), ref["thr_val"])
    assert np.array_equal(got["thr_idx"], ref["thr_idx"])
    assert np.all(got["alpha_is_upper"] == 1)
    assert np.allclose(got["alpha"], ref["alpha"], rtol=gu.AB_RTOL, atol=0) and np.array_equal(got["beta"], -got["alpha"])
    if n < 2:
        return                             # the packer and the layers need two weights
    # the same packing kernel turns the descriptor into the sign mask
    E, ecnt = dab.dab_pack_weights(gu.to_gpu(W.reshape(F, n, 1, 1)), out["thr_val"], out["thr_idx"], out["alpha_is_upper"])
    torch.cuda.synchronize()
    E_ref, ecnt_ref = opk.pack_weights(ref["e"].reshape(F, n, 1, 1))
    assert np.array_equal(gu.u32(E), E_ref) and np.array_equal(gu.u32(ecnt), ecnt_ref)
    # a fully-connected layer on these weights: y = alpha * (2 * #agreements - n), XNOR-Net's form
    B = 9
    x = rng.standard_normal((B, n)).astype(np.float32)
    A = dab.dab_pack_activations(gu.to_gpu(x), dab.DAB_LAYOUT_NHWC, None).reshape(B, -1)
    Y, s1 = dab.dab_binfc(A, E, out["alpha"], out["beta"], n, want_s1=True)
    torch.cuda.synchronize()
    a = olay.binarize_activations(x)
    b = np.where(W >= 0, 1, -1)
    agree = (a[:, None, :] == b[None, :, :]).sum(axis=2)
    y_ref = got["alpha"].astype(np.float64)[None, :] * (2 * agree - n)
    tol = gu.Y_RTOL * np.maximum(np.abs(y_ref), got["alpha"].astype(np.float64)[None, :] * n)
    assert np.all(np.abs(Y.cpu().numpy() - y_ref) <= tol)


# (name, B, C, H, W, F, k, pad, stride): padding as wide as the kernel or wider, on each of the product kernels
# (that a layer takes the kernel it is named after is checked on the CPU, test_host_sanitizers.py)
BORDER_LAYERS = [("persistent k1p1", 120, 64, 12, 13, 64, 1, 1, 1), ("persistent k2p2", 150, 64, 12, 13, 64, 2, 2, 1),
                 ("persistent k3p3", 150, 96, 9, 8, 100, 3, 3, 1), ("persistent k1p2s2", 200, 128, 9, 9, 130, 1, 2, 2),
                 ("block k1p1", 1, 64, 6, 6, 32, 1, 1, 1), ("block k2p3", 2, 33, 5, 5, 7, 2, 3, 1),
                 ("block k1p1, 40 blocks", 6, 64, 12, 13, 64, 1, 1, 1), ("block k2p2", 6, 64, 12, 13, 64, 2, 2, 1),
                 ("block k3p3", 5, 96, 9, 8, 100, 3, 3, 1), ("block k1p2s2", 40, 128, 9, 9, 130, 1, 2, 2),
                 ("split k1p1", 64, 4096, 8, 8, 512, 1, 1, 1), ("workspace k6p6", 30, 64, 8, 8, 100, 6, 6, 1)]


@pytest.mark.parametrize("case", BORDER_LAYERS, ids=lambda c: c[0])
def test_padding_that_reaches_the_kernel_extent(case):
    """Windows that lie entirely in the zero border: s1 = sA = 0 there, everything else as usual."""
    import zlib
    name, B, C, H, W, F, k, p, s = case
    L = Layer(name, C=C, H=H, W=W, F=F, kh=k, kw=k, pad=p, stride=s)
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    x = rng.standard_normal((B, C, H, W)).astype(np.float32)
    w = (0.05 * rng.standard_normal((F, C, k, k)) + 0.01).astype(np.float32)
    gu.check_layer(L, x, w, tau=None)
