"""Whether an object's batches are sorted by default, through lsnif_get_tuning, lsnif_set_tuning and
the cache: reading a tuning and setting it again, and a pair autotune, choose no sort."""
import json

import numpy as np
import pytest

import workloads as W
from tests.test_gpu_tuning import L   # noqa: F401

pytestmark = pytest.mark.gpu


def sort_ms(L, ctx, oid, rays, out):   # noqa: F811
    """Milliseconds that a query of the object spends in the coherence sort's place."""
    import torch
    for _ in range(3):
        L.lsnif_query(ctx, oid, rays, out)
    torch.cuda.synchronize()
    L.lsnif_profile_enable(ctx, True)
    for _ in range(8):
        L.lsnif_query(ctx, oid, rays, out)
    ms, _, _, k = L.lsnif_profile_read(ctx)
    L.lsnif_profile_enable(ctx, False)
    return ms / k


def test_default_sort_survives_get_set_and_cache(L, tmp_path):   # noqa: F811
    import torch
    small, large = W.configs.c1_object(), W.configs.c2_object()   # tables of 512 KiB and 32 MiB in FP16
    rays_np = W.sphere_to_box_rays(np.random.default_rng(5), 200_000, radius=2.0, half_box=1.0)
    rays = torch.from_numpy(rays_np).cuda()
    out = torch.empty((len(rays_np), 6), dtype=torch.float32, device="cuda")
    path = str(tmp_path / "tune.json")
    ctx = L.lsnif_create(0, autotune_cache=path)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(small, "fp16", "fp16"))
        t = L.lsnif_get_tuning(ctx, oid)
        none = sort_ms(L, ctx, oid, rays, out)
        L.lsnif_set_tuning(ctx, oid, **{**t, "sort_bits": 5})
        full = sort_ms(L, ctx, oid, rays, out)
        print("sort: none", none, "set", full, flush=True)
        assert none < full / 2                        # an unset object is not sorted, a set one is
        assert L.lsnif_get_tuning(ctx, oid)["sort_bits"] == 5
        # what an untouched object reports can be set again
        oid = L.lsnif_build(ctx, L.ObjectDesc(small, "fp16", "fp16"))
        t = L.lsnif_get_tuning(ctx, oid)
        assert t["sort_bits"] == 0
        L.lsnif_set_tuning(ctx, oid, **{**t, "walk_chunks": 2})
        assert sort_ms(L, ctx, oid, rays, out) < full / 2
        big = L.lsnif_build(ctx, L.ObjectDesc(large, "fp16", "fp16"))
        assert L.lsnif_get_tuning(ctx, big)["sort_bits"] == 5
    finally:
        L.lsnif_destroy(ctx)
    # a pair autotune chooses no sort, in this context or in one that reads its cache
    ctx = L.lsnif_create(0, autotune_cache=path)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(small, "fp16", "fp16"))
        eye = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
        inst = torch.from_numpy(L.instances_array([(oid, eye)])).cuda()
        pr = torch.arange(len(rays_np), dtype=torch.int32, device="cuda")
        best = L.lsnif_autotune_pairs(ctx, rays, pr, torch.zeros_like(pr), inst, out)
        assert L.lsnif_get_tuning(ctx, oid) == best and best["sort_bits"] == 0
        assert sort_ms(L, ctx, oid, rays, out) < full / 2
    finally:
        L.lsnif_destroy(ctx)
    (entry,) = json.load(open(path))["entries"].values()
    assert entry == best
    ctx = L.lsnif_create(0, autotune_cache=path)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(small, "fp16", "fp16"))
        assert L.lsnif_get_tuning(ctx, oid) == best
        assert sort_ms(L, ctx, oid, rays, out) < full / 2
    finally:
        L.lsnif_destroy(ctx)
