"""Pair preparation and coherence sort at the sizes where their passes change: each pair's answer
is the single-object query's, whatever path grouped it."""

import numpy as np
import pytest

from paper_2504_21627_amd import lsnif as L

pytestmark = pytest.mark.gpu


def build(ctx, count, seed=0):
    from tests.test_oracle_pins import tiny_object
    rng = np.random.default_rng(seed)
    return [L.lsnif_build(ctx, L.ObjectDesc(tiny_object(8, rng.uniform(size=512) < 0.3, H=4, L=1, F=2, R=[8], log2_T=8,
                                                        width=64, n_hidden=1, seed=i), "fp16", "fp16"))
            for i in range(count)]


# objects in the table, pair_bits of each: keys of 12 to 25 bits, up to and past 1,023 objects
@pytest.mark.parametrize("count,bits", [(1, 1), (5, 4), (5, 6), (65, 3), (65, 6), (1100, 1)])
def test_pairs_at_the_switches(count, bits):
    import torch
    torch.cuda.init()
    rng = np.random.default_rng(count)
    ctx = L.lsnif_create(0)
    try:
        ids = build(ctx, count)
        for i in ids[::3]:
            L.lsnif_set_tuning(ctx, i, 5, bits, 0)
        used = [ids[0], ids[-1], ids[len(ids) // 2]]
        gone = ids[len(ids) // 3] if count > 3 else None
        if gone in used:
            gone = None
        if gone is not None:
            L.lsnif_release(ctx, gone)
        eye = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
        insts = [(i, eye) for i in used] + [(10 ** 6, eye)] + ([(gone, eye)] if gone is not None else [])
        inst = torch.from_numpy(L.instances_array(insts)).cuda()
        top = 262145
        o = rng.uniform(-1.2, 1.2, (top, 3))
        d = rng.standard_normal((top, 3))
        rays = torch.from_numpy(np.concatenate([o, d, np.zeros((top, 1)), np.full((top, 1), np.inf)], 1)
                                .astype(np.float32)).cuda()
        owner = torch.from_numpy(rng.integers(0, len(insts) + 2, top).astype(np.int32)).cuda()   # 2 of no instance
        want = torch.empty((len(used), top, 6), dtype=torch.float32, device="cuda")
        for k, i in enumerate(used):
            L.lsnif_query(ctx, i, rays, want[k])
        miss = torch.zeros(6, device="cuda")
        miss[1], miss[5:] = float("inf"), torch.tensor([-1], dtype=torch.int32, device="cuda").view(torch.float32)
        for n in (1, 255, 257, 2048, 8192, 8193, 20000, 262144, 262145):
            pr = torch.randperm(n, device="cuda").int()
            pi = owner[:n][pr.long()].contiguous()
            out = torch.full((n, 6), -7.0, device="cuda")
            L.lsnif_query_pairs(ctx, rays[:n], pr, pi, inst, out)
            torch.cuda.synchronize()
            ref = miss.expand(n, 6).clone()
            for k in range(len(used)):
                sel = owner[:n] == k
                ref[sel] = want[k, :n][sel]
            cols = [0, 1, 5]   # world normals are renormalised
            assert torch.equal(out[:, cols].view(torch.int32), ref[:, cols].view(torch.int32)), n
            assert torch.allclose(out[:, 2:5], ref[:, 2:5], atol=1e-6), n
            if n > 1000:
                assert int((out[:, 0].view(torch.int32) == 1).sum()) > n // 50
    finally:
        L.lsnif_destroy(ctx)


@pytest.mark.parametrize("n", [8192, 16383, 262144, 262145])
def test_sorted_batches_at_the_switches(n):
    """Two 10-bit passes (sort_bits 1..5, up to 262,144 rays) and the 8-bit ones answer alike."""
    import torch
    torch.cuda.init()
    rng = np.random.default_rng(n)
    ctx = L.lsnif_create(0)
    try:
        oid = build(ctx, 1)[0]
        rays = torch.from_numpy(np.concatenate([rng.uniform(-1.2, 1.2, (n, 3)), rng.standard_normal((n, 3)),
                                                np.zeros((n, 1)), np.full((n, 1), np.inf)], 1).astype(np.float32)).cuda()
        ref = None
        for sb in (0, 1, 2, 5, 6, 7):
            L.lsnif_set_tuning(ctx, oid, sb, 4, 0)
            out = torch.full((n, 6), float("nan"), device="cuda")
            L.lsnif_query(ctx, oid, rays, out)
            torch.cuda.synchronize()
            ref = out if ref is None else ref
            assert torch.equal(out.view(torch.int32), ref.view(torch.int32)), sb
    finally:
        L.lsnif_destroy(ctx)


@pytest.mark.parametrize("n_rays,n_inst", [(1, 1), (1023, 7), (1024, 8), (1025, 9), (3000, 256), (3000, 257)])
def test_broad_phase_at_the_switches(n_rays, n_inst):
    """The pairs by masks (at most 256 instances) and without, against the pair query's own slab
    test: a pair is listed iff its ray meets the instance's grid, by ray, then instance."""
    import torch
    import oracle
    from tests.scene import small_scene
    torch.cuda.init()
    objs, insts, _, rays_np = small_scene()
    rays_np = np.resize(rays_np, (n_rays, 8)).astype(np.float32)
    ctx = L.lsnif_create(0)
    try:
        ids = [L.lsnif_build(ctx, L.ObjectDesc(ob, "fp16", "fp16")) for ob in objs]
        many = [insts[k % len(insts)] for k in range(n_inst)]
        inst = torch.from_numpy(L.instances_array([(ids[k], m) for k, m in many])).cuda()
        rays = torch.from_numpy(rays_np).cuda()
        pr = torch.empty(n_rays * n_inst, dtype=torch.int32, device="cuda")
        pi = torch.empty_like(pr)
        c = L.lsnif_broad_phase(ctx, rays, inst, pr, pi)
        torch.cuda.synchronize()
        got = pr[:c].cpu().numpy().astype(np.int64) * n_inst + pi[:c].cpu().numpy()
        wr, wi = oracle.broad_phase(objs, many, rays_np)[:2]
        want = np.asarray(wr, np.int64) * n_inst + np.asarray(wi, np.int64)
        assert np.array_equal(got, np.sort(want))
    finally:
        L.lsnif_destroy(ctx)
