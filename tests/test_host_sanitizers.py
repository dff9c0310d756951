"""The library's host code (geometry checks, planners, workspace sizes, argument validation) built with
AddressSanitizer and UBSan (host side of the hipcc compile only) and driven over random layer
geometries by tests/host/fuzz_plans.cpp, which also checks the invariants the kernels rely on.
No GPU is needed: every entry point ends before its first launch here."""
import os
import subprocess

import pytest

from paper_1804_02941_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def fuzz(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "fuzz_plans")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC") and not f.startswith("-Rpass")]
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-g",
           "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
           "-Xarch_host", "-fno-sanitize-recover=undefined",
           "-I", os.path.join(ROOT, "include"), "-I", build.CSRC,
           *[os.path.join(build.CSRC, s) for s in build.SOURCES],
           os.path.join(ROOT, "tests", "host", "fuzz_plans.cpp"), "-o", exe]
    p = subprocess.run(cmd, capture_output=True, text=True)
    assert p.returncode == 0, p.stdout[-3000:] + p.stderr[-3000:]
    return exe


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_geometries_through_the_host_code(fuzz, seed):
    p = subprocess.run([fuzz, "100000", str(seed)], capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stdout[-2000:] + p.stderr[-4000:]
    assert "geometries checked" in p.stdout


def routes(fuzz, layers, mode="route"):
    """[(kernel of the fp32 form, of the packed-sign form)] of layers (B, C, H, W, F, k, pad, stride)."""
    args = [str(v) for B, C, H, W, F, k, p, s in layers for v in (B, C, H, W, F, k, k, p, p, s, s)]
    out = subprocess.run([fuzz, mode, *args], capture_output=True, text=True, check=True).stdout
    return [tuple(line.split()) for line in out.splitlines()]


def test_long_reductions_take_the_kernel_that_measured_faster(fuzz):
    """Layers whose times in the three forms differ by more than a fifth."""
    layers = {
        "expanded": [(34, 992, 52, 52, 512, 5, 2, 1), (102, 832, 21, 22, 640, 7, 0, 1)],
        "block": [(1, 768, 47, 47, 384, 3, 0, 1), (23, 222, 31, 8, 464, 5, 2, 2), (80, 395, 7, 7, 140, 3, 1, 1)],
        "split": [(1024, 9216, 1, 1, 4096, 1, 0, 1), (1024, 4096, 1, 1, 4096, 1, 0, 1), (64, 512, 7, 7, 512, 3, 1, 1),
                  (789, 8296, 1, 1, 928, 1, 0, 1), (25, 487, 23, 27, 379, 3, 1, 2), (2, 184, 48, 46, 224, 5, 2, 1),
                  (112, 720, 54, 10, 74, 7, 0, 1), (64, 138, 48, 10, 816, 7, 0, 1)],
    }
    for kernel, ls in layers.items():
        assert routes(fuzz, ls) == [(kernel, kernel)] * len(ls)


def test_fp32_outputs_of_more_filters_than_its_row_offsets_reach_leave_the_persistent_kernel(fuzz):
    wide = [(B, 64, 1, 1, F, 1, 0, 1) for B, F in ((1, 1 << 24), (1, (1 << 24) + 1), (2, 18400000), (29, 18400000))]
    assert routes(fuzz, wide) == [("direct", "direct")] + [("split", "direct")] * 3


# The persistent kernel's outputs: what reads one of up to 96 MB finds it in the memory-side cache.
STORES = {
    "through": [(64, 64, 56, 56, 64, 3, 1, 1), (255, 256, 15, 15, 256, 3, 1, 1), (200, 64, 35, 35, 128, 5, 0, 1), (52, 128, 28, 28, 512, 1, 0, 1),
                (98303, 320, 1, 1, 256, 1, 0, 1), (98304, 320, 1, 1, 256, 1, 0, 1), (200000, 320, 1, 1, 132, 1, 0, 1)],
    "streamed": [(98305, 320, 1, 1, 256, 1, 0, 1), (256, 64, 35, 35, 128, 5, 0, 1), (170001, 320, 1, 1, 160, 1, 0, 1)],
    "plain": [(19044, 320, 1, 1, 290, 1, 0, 1), (200000, 320, 1, 1, 133, 1, 0, 1)],
}


@pytest.mark.parametrize("policy", STORES)
def test_outputs_that_the_memory_side_cache_holds_are_not_streamed(fuzz, policy):
    assert routes(fuzz, STORES[policy], "plan") == [("direct", policy)] * len(STORES[policy])


def test_the_gpu_tests_of_the_long_reduction_kernels_reach_them(fuzz):
    from test_gpu_rebinarize import EXPANDED_LAYERS, SPLIT_LAYERS
    for layers, kernel in ((SPLIT_LAYERS, "split"), (EXPANDED_LAYERS, "expanded")):
        for layer, r in zip(layers, routes(fuzz, [c[1:] for c in layers])):
            assert r == (kernel, kernel), layer[0]


def test_the_gpu_tests_of_shares_reach_the_exchanges_they_name(fuzz):
    """Every kernel of the case lists with the shares, the exchange and the stores that the list is for."""
    from test_gpu_rebinarize import SPLIT_LAYERS
    from test_gpu_share_exchange import CASES
    for name, cases in CASES.items():
        for case, plan in zip(cases, routes(fuzz, [(B, K, 1, 1, F, 1, 0, 1) for B, K, F in cases], "plan")):
            assert set(name.split()) <= set(plan), case
    for layer, plan in zip(SPLIT_LAYERS, routes(fuzz, [c[1:] for c in SPLIT_LAYERS], "plan")):
        words, shares = layer[0].split("_")[:2]
        assert plan[:3] == ("split", words, shares) and plan[3] == ("alone" if shares == "s1" else "16-bit"), layer[0]


def test_the_gpu_tests_of_wide_padding_reach_the_kernels_they_name(fuzz):
    from test_gpu_parity import BORDER_LAYERS
    kernels = {"persistent": "direct", "block": "block", "split": "split", "workspace": "expanded"}
    for layer, r in zip(BORDER_LAYERS, routes(fuzz, [c[1:] for c in BORDER_LAYERS])):
        assert r == (kernels[layer[0].split()[0]],) * 2, layer[0]


def test_the_gpu_tests_of_the_weights_only_layer_reach_the_forms_they_name(fuzz):
    from test_gpu_wbin_forms import LAYERS
    args = [str(v) for _, (B, C, H, W, F, k, p, s) in LAYERS for v in (B, C, H, W, F, k, k, p, p, s, s)]
    out = subprocess.run([fuzz, "wbin", *args], capture_output=True, text=True, check=True).stdout.split()
    for (form, layer), got in zip(LAYERS, out, strict=True):
        assert tuple(int(v) for v in got.split(",")) == form, layer


# Large layers timed in every form (us: the patch kernel's 4,4 | the direct kernel's 32,4,1): 165 | 192, 160 | 190, 88.9 | 99.6.
LARGE_WBIN = [((256, 256, 15, 15, 256, 3, 1, 1), (0, 4, 4)), ((256, 256, 14, 14, 256, 3, 1, 1), (0, 4, 4)),
              ((128, 256, 15, 15, 256, 3, 1, 1), (0, 4, 4))]


def test_large_weights_only_layers_take_the_form_measured_fastest(fuzz):
    args = [str(v) for (B, C, H, W, F, k, p, s), _ in LARGE_WBIN for v in (B, C, H, W, F, k, k, p, p, s, s)]
    out = subprocess.run([fuzz, "wbin", *args], capture_output=True, text=True, check=True).stdout.split()
    assert [tuple(int(v) for v in got.split(",")) for got in out] == [form for _, form in LARGE_WBIN]
