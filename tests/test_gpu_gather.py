"""The gather-ceiling kernel takes the query's own split of the gathers: no longer than the query kernel on
the same batch, and each ray's sum is that of the oracle's encoding row, also with 3 features per
level (4 corners on aligned levels), with a tile's points in several passes and with ragged tiles."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2504_21627_amd import lsnif as L
from tests.test_gpu_query_tiles import U

pytestmark = pytest.mark.gpu

# feat, mlp, F, L, H, levels aligned with the faces
CASES = [("fp32", "fp32", 3, 4, 18, "all"), ("fp16", "fp16", 3, 3, 18, "even"), ("bf16", "bf16", 3, 5, 64, "all"),
         ("fp16", "fp16", 2, 9, 64, ""), ("fp32", "fp32", 2, 32, 18, "")]


@pytest.mark.parametrize("feat,mlp,F,levels,H,aligned", CASES)
def test_sums(feat, mlp, F, levels, H, aligned):
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(levels)
    V = 16
    R = [max(1, 5 * (l + 1)) for l in range(levels)]
    if aligned:
        R = [V * (l + 1) + (0 if aligned == "all" or l % 2 == 0 else 1) for l in range(levels)]
    obj = tiny_object(V, rng.uniform(size=V ** 3) < 0.8, H=H, L=levels, F=F, R=R, log2_T=9, width=64, n_hidden=1, seed=2)
    rays = adversarial_rays(rng, V, n_random=500).astype(np.float32)
    o = oracle.query(obj, rays, debug=True)
    want, scale = o["enc"].sum(1), np.abs(o["enc"]).sum(1)
    assert (o["count"] > 12).sum() > 50
    ctx = L.lsnif_create(0)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(obj, feat, mlp))
        for n in (1, 63, 64, 65, len(rays)):
            sums = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
            L.lsnif_gather_ceiling(ctx, oid, torch.from_numpy(rays[:n]).cuda(), sums)
            torch.cuda.synchronize()
            got = sums.cpu().numpy().astype(np.float64)
            # the features' rounding, and the float32 sum of H L F of them
            tol = (max(4 * U[feat], 1e-5) + 2.0 ** -24 * H * levels * F) * scale[:n] + 1e-30
            assert np.all(np.abs(got - want[:n]) <= tol), (n, float(np.abs(got - want[:n]).max()))
    finally:
        L.lsnif_destroy(ctx)


def kernel_ms(ctx, call):
    import torch
    for _ in range(3):
        call()
    torch.cuda.synchronize()
    L.lsnif_profile_enable(ctx, True)
    for _ in range(10):
        call()
    _, _, ms, k = L.lsnif_profile_read(ctx)
    L.lsnif_profile_enable(ctx, False)
    return ms / k


@pytest.mark.parametrize("which", ["paper", "c2"])
def test_takes_no_longer_than_the_query(which):
    import torch
    if which == "paper":   # 3 features per level, both levels aligned
        obj = W.configs.paper_object(seed=1)
        rays_np = W.sphere_to_box_rays(np.random.default_rng(1), 1 << 20, radius=2.0, half_box=1.0)
    else:
        obj, rays_np = W.configs.c2_object(), W.configs.subsample(W.configs.c2_rays(), 300000, seed=1)
    rays = torch.from_numpy(rays_np).cuda()
    out = torch.empty((len(rays_np), 6), dtype=torch.float32, device="cuda")
    sums = torch.empty(len(rays_np), dtype=torch.float32, device="cuda")
    ctx = L.lsnif_create(0)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(obj, "fp16", "fp16"))
        query = kernel_ms(ctx, lambda: L.lsnif_query(ctx, oid, rays, out))
        gather = kernel_ms(ctx, lambda: L.lsnif_gather_ceiling(ctx, oid, rays, sums))
        print(which, "query", query, "gathers alone", gather, "ms", flush=True)
        assert gather < query
    finally:
        L.lsnif_destroy(ctx)
