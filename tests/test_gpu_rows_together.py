"""Weight sides of short and of long rows in one call: one launch up to 5120 rows (and 200 MB of packing beside it), two beyond.  Either
way the results are those of the separate calls, bit for bit."""
import pytest
import torch

from paper_1804_02941_amd import binding as dab

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# (F, C, k) of the layers: rows of up to 2304 weights, of 4609 to 9216 and of 9217 to 13312 (and one class between)
@pytest.mark.parametrize("layers", [
    [(70, 64, 1), (33, 4700, 1)], [(3, 256, 3), (65, 9216, 1)], [(1, 2, 1), (1, 13312, 1)], [(130, 30, 5), (64, 256, 7), (9, 9217, 1)],
    [(512, 2304, 1), (40, 1024, 3), (20, 4608, 1)],         # a layer of the class between
    [(5056, 20, 1), (64, 4700, 1)], [(5057, 20, 1), (64, 4700, 1)],         # the last in one launch, the first in two
], ids=str)
@pytest.mark.parametrize("pack", [False, True])
def test_short_and_long_rows(layers, pack):
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(F * C for F, C, _ in layers))
    items, ref = [], []
    for F, C, k in layers:
        W = torch.randn(F, C, k, k, generator=g, device=DEV)
        if C * k * k > 9000:
            W.view(F, -1)[0, :4300] = 0.0                           # a bucket of more elements than it counts: sorted
        items.append(dict(W=W, est=dab.estimate_outputs(F, DEV), packed=dab.pack_weights_outputs(F, C, k, k, DEV)))
        est = dab.dab_estimate_alpha_beta(W.view(F, -1))
        ref.append((est, dab.dab_pack_weights(W, est["thr_val"], est["thr_idx"], est["alpha_is_upper"])))
    jobs = dab.weight_jobs(items)
    if pack:
        X = torch.randn(5, 9, 7, 70, generator=g, device=DEV)
        A = torch.empty((5, 9, 7, 3), dtype=torch.int32, device=DEV)
        dab.dab_prepare_layers(jobs, dab.pack_jobs([(X, None, A)]))
        assert torch.equal(A, dab.dab_pack_activations(X))
    else:
        dab.dab_binarize_weights_multi(jobs)
    for it, (est, packed) in zip(items, ref):
        for key in est:
            assert torch.equal(it["est"][key], est[key]), key
        assert torch.equal(it["packed"][0], packed[0]) and torch.equal(it["packed"][1], packed[1])


# The same classes with rows of a few distinct values, which the bucket search leaves to the sort kernel: first, last and
# neighbouring filters of every layer, short rows among them.
@pytest.mark.parametrize("layers", [
    [(70, 2304, 1), (33, 4700, 1)], [(65, 256, 3), (40, 1024, 3)], [(64, 1500, 1), (9, 13312, 1)], [(130, 90, 5), (17, 9000, 1), (9, 9217, 1)],
], ids=str)
@pytest.mark.parametrize("bounded", [False, True])
def test_rows_handed_over_to_the_sort(layers, bounded):
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(F * C for F, C, _ in layers))
    items, ref, coarse = [], [], []
    for F, C, k in layers:
        n = C * k * k
        W = torch.randn(F, C, k, k, generator=g, device=DEV)
        few = sorted({0, 1, F // 2, F - 1})
        W.view(F, n)[few] = torch.round(W.view(F, n)[few] + 0.3)
        est = dab.dab_estimate_alpha_beta(W.view(F, n))
        prev = None
        if bounded:
            prev = est["K"].clone(), est["alpha_is_upper"].clone(), n // 3
            est = dab.dab_estimate_alpha_beta_bounded(W.view(F, n), *prev)
        items.append(dict(W=W, est=dab.estimate_outputs(F, DEV), packed=dab.pack_weights_outputs(F, C, k, k, DEV), prev=prev))
        ref.append((est, dab.dab_pack_weights(W, est["thr_val"], est["thr_idx"], est["alpha_is_upper"])))
        coarse.append(few)
    jobs = dab.weight_jobs(items)
    ws = torch.full((dab.lib().dab_binarize_weights_multi_workspace_bytes(jobs, len(jobs)),), 255, dtype=torch.uint8, device=DEV)
    assert ws.numel() == sum((F + 255) // 256 * 256 for F, _, _ in layers)
    dab.dab_binarize_weights_multi(jobs, ws=ws)
    for (F, _, _), flags, few, it, (est, packed) in zip(layers, ws.split([(F + 255) // 256 * 256 for F, _, _ in layers]), coarse, items, ref):
        assert set(few) <= set(flags[:F].nonzero().flatten().tolist()) and int(flags[:F].sum()) < F        # (the others were finished)
        for key in est:
            assert torch.equal(it["est"][key], est[key]), key
        assert torch.equal(it["packed"][0], packed[0]) and torch.equal(it["packed"][1], packed[1])
