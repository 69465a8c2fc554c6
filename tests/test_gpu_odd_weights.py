"""Weights and table entries that are not finite.  Weights on inputs of the later boundary points: a ray
that lists few voxels does not use them, and its answer does not depend on the rays beside it."""
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
    odd.weights[0][::3, 6 * levels * F:] = np.nan
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


@pytest.mark.parametrize("feat,mlp", [("fp32", "fp32"), ("fp16", "fp16"), ("bf16", "fp32")])
def test_infinite_entries_on_aligned_levels(feat, mlp):
    """Three features per level: a level aligned with the voxel faces gives the features that it gives
    beside one that is not aligned, infinities included (the sums over a face's 4 corners and
    over all 8, of which 4 weigh nothing)."""
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(11)
    V = 16
    occ = rng.uniform(size=V ** 3) < 0.4
    rays = adversarial_rays(rng, V, n_random=600).astype(np.float32)
    enc = []
    ctx = L.lsnif_create(0)
    try:
        for last in (2 * V, 2 * V + 1):
            obj = tiny_object(V, occ, H=18, L=2, F=3, R=[V, last], log2_T=13, width=64, n_hidden=2, seed=4)
            at = np.random.default_rng(5).integers(1, 1 << 13, 600)
            obj.tables[0, at, at % 3] = np.where(at & 4, np.inf, -np.inf)
            oid = L.lsnif_build(ctx, L.ObjectDesc(obj, feat, mlp))
            enc.append(run_enc(ctx, oid, obj, rays)[:, :, 0, :])
    finally:
        L.lsnif_destroy(ctx)
    print(feat, mlp, "infinite features", int(np.isinf(enc[1]).sum()), "not a number", int(np.isnan(enc[1]).sum()), flush=True)
    assert np.isinf(enc[1]).sum() > 500
    assert np.array_equal(enc[0], enc[1], equal_nan=True)


def run_enc(ctx, oid, obj, rays):
    import torch
    n = len(rays)
    r = torch.from_numpy(rays).cuda()
    out = torch.empty((n, 6), dtype=torch.float32, device="cuda")
    enc = torch.zeros((n, obj.H * obj.L * obj.F), dtype=torch.float32, device="cuda")
    L.lsnif_query_debug(ctx, oid, r, out, {"enc": enc})
    torch.cuda.synchronize()
    return enc.cpu().numpy().reshape(n, obj.H, obj.L, obj.F)
