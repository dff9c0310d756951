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
