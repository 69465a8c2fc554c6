"""Weights that are not finite, on inputs of the later boundary points: a ray that lists few voxels
does not use them, and its answer does not depend on the rays beside it."""
import copy

import numpy as np
import pytest

import oracle
from paper_2504_21627_amd import lsnif as L
from tests.test_gpu_query_tiles import run

pytestmark = pytest.mark.gpu

# feat, mlp, F, L, width, H: 16, 32 and 64 rays per block by the batch sizes below
CASES = [("fp32", "fp32", 2, 4, 64, 18), ("fp32", "fp32", 3, 2, 128, 18), ("fp16", "fp32", 2, 9, 64, 64),
         ("fp16", "fp16", 2, 4, 64, 18), ("fp16", "fp16", 3, 2, 128, 18), ("fp32", "bf16", 2, 4, 64, 64)]


@pytest.mark.parametrize("feat,mlp,F,levels,width,H", CASES)
def test_short_rays_do_not_meet_the_weights_of_later_points(feat, mlp, F, levels, width, H):
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(9)
    V = 16
    obj = tiny_object(V, rng.uniform(size=V ** 3) < 0.3, H=H, L=levels, F=F, R=[5 * (l + 1) for l in range(levels)],
                      log2_T=9, width=width, n_hidden=2, seed=3)
    odd = copy.copy(obj)
    odd.weights = [w.copy() for w in obj.weights]
    odd.weights[0][:, 4 * levels * F:] = 1e30 if mlp == "fp16" else np.inf   # rounds to an infinity in FP16
    base = adversarial_rays(rng, V, n_random=400).astype(np.float32)
    count = oracle.query(obj, base, debug=True)["count"]
    assert (count == 4).sum() > 10 and (count > 8).sum() > 40
    ctx = L.lsnif_create(0)
    try:
        ids = [L.lsnif_build(ctx, L.ObjectDesc(o, feat, mlp)) for o in (obj, odd)]
        for n in (len(base), 20000, 400000 if mlp == "fp32" else 40000):
            at = np.arange(n) % len(base)
            short = count[at] <= 4
            want, got = (run(ctx, i, obj, base[at]) for i in ids)
            for k in want:
                a, b = want[k][short].view(np.uint32), got[k][short].view(np.uint32)
                print(feat, mlp, width, n, k, int((a != b).any(axis=1).sum()), "of", int(short.sum()), flush=True)
                assert np.array_equal(a, b), (k, n)
    finally:
        L.lsnif_destroy(ctx)
