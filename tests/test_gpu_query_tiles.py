"""The query kernel at the edges of its tiles: batch sizes around 16, 32 and 64 rays per block
and the switches between them, level counts that leave a batch of levels partly empty, point
caps that need several passes over the tile's points, every MLP type and both widths.

Small batches against the oracle (raw outputs within the forward-error bound of the type, as
the parity tests); larger ones hold the same rays again, whose answers must be the same bits."""

import numpy as np
import pytest

import oracle
from paper_2504_21627_amd import lsnif as L
from tests.parity import output_bound

pytestmark = pytest.mark.gpu

U = {"fp32": 2.0 ** -24, "fp16": 2.0 ** -11, "bf16": 2.0 ** -8, "fp8": 2.0 ** -4}

# feat, mlp, F, L, width, H, V, density of occupied voxels[, the levels aligned with the faces]
CASES = [("fp32", "fp32", 2, 1, 64, 18, 8, 0.5), ("fp32", "fp32", 3, 5, 128, 18, 16, 0.5),
         ("fp16", "fp32", 2, 9, 64, 64, 32, 0.9), ("fp32", "fp32", 3, 32, 64, 18, 8, 0.4),
         ("fp16", "fp16", 2, 1, 64, 2, 8, 0.5), ("fp16", "fp16", 2, 5, 64, 18, 16, 0.3),
         ("fp16", "fp16", 3, 3, 128, 18, 16, 0.5), ("bf16", "bf16", 2, 13, 64, 64, 32, 0.9),
         ("fp32", "fp16", 2, 16, 128, 18, 16, 0.2), ("fp16", "fp16", 3, 32, 64, 18, 8, 0.4),
         ("fp16", "fp8", 2, 7, 64, 18, 16, 0.5), ("bf16", "fp8", 3, 5, 128, 18, 16, 0.5),
         ("fp16", "fp16", 3, 3, 128, 18, 16, 0.5, "all"), ("fp32", "fp32", 3, 3, 64, 18, 16, 0.5, "all"),
         ("fp16", "fp16", 3, 4, 64, 18, 16, 0.5, "even"), ("bf16", "fp32", 3, 4, 128, 18, 16, 0.5, "even")]
CASES = [c if len(c) == 9 else c + ("",) for c in CASES]


def run(ctx, oid, obj, rays, enc=False):
    import torch
    n = len(rays)
    r = torch.from_numpy(np.ascontiguousarray(rays, np.float32)).cuda()
    out = torch.empty((n, 6), dtype=torch.float32, device="cuda")
    bufs = {"out": torch.zeros((n, obj.out_dim), dtype=torch.float32, device="cuda")}
    if enc:
        bufs["enc"] = torch.zeros((n, obj.H * obj.L * obj.F), dtype=torch.float32, device="cuda")
    L.lsnif_query_debug(ctx, oid, r, out, bufs)
    plain = torch.empty_like(out)
    L.lsnif_query(ctx, oid, r, plain)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), plain.view(torch.int32))
    return {"hits": out.cpu().numpy(), **{k: v.cpu().numpy() for k, v in bufs.items()}}


@pytest.mark.parametrize("feat,mlp,F,levels,width,H,V,density,aligned", CASES)
def test_tile_edges(feat, mlp, F, levels, width, H, V, density, aligned):
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(levels * 7 + H)
    occ = rng.uniform(size=V ** 3) < density
    R = [max(1, int(V * (l + 1) / 3)) for l in range(levels)]
    if aligned:
        R = [V * (l + 1) + (0 if aligned == "all" or l % 2 == 0 else 1) for l in range(levels)]
    obj = tiny_object(V, occ, H=H, L=levels, F=F, R=R, log2_T=9, width=width, n_hidden=2, seed=levels)
    obj.tables *= np.float32(1e-2)
    base = adversarial_rays(rng, V, n_random=400).astype(np.float32)
    print(f"tiles {feat}/{mlp} F={F} L={levels} width={width} H={H}: {len(base)} rays", flush=True)
    scale = [1e-2 / 448] + [4e-2 / 448] * 2 if mlp == "fp8" else None
    ctx = L.lsnif_create(0)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(obj, feat, mlp, scale))
        ref = run(ctx, oid, obj, base, enc=True)
        if mlp != "fp8":
            o = oracle.query(obj, base, debug=True)
            u = max(U[feat], U[mlp])
            cand = o["count"] > 0
            assert cand.sum() > 100
            err = np.abs(ref["out"][cand].astype(np.float64) - o["out"][cand])
            bound = output_bound(obj, o["enc"], u)[cand]
            assert np.all(err <= 4 * bound + 1e-30), float((err / np.maximum(bound, 1e-30)).max())
        per = H * levels * F
        for n in (1, 15, 16, 17, 31, 33, 64, 65, 8192, 8193, 32768, 32769, 393217, 786433):
            small = n * per < 1 << 28
            got = run(ctx, oid, obj, np.resize(base, (n, 8)), enc=small)
            for k in got:
                want = np.resize(ref[k], (n,) + ref[k].shape[1:])
                assert got[k].tobytes() == want.tobytes(), (n, k)
    finally:
        L.lsnif_destroy(ctx)


@pytest.mark.parametrize("feat,mlp,F,width", [("fp16", "fp16", 2, 64), ("fp32", "fp32", 3, 128)])
def test_pairs_of_objects_with_other_level_counts(feat, mlp, F, width):
    """One pair launch over objects whose points take 1 to 4 batches of levels: each ray's hit
    is the single-object query's."""
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(3)
    objs = []
    for i, (levels, H) in enumerate([(1, 18), (5, 4), (9, 18), (13, 32)]):
        occ = rng.uniform(size=16 ** 3) < 0.4
        objs.append(tiny_object(16, occ, H=H, L=levels, F=F, R=[8 + 4 * l for l in range(levels)], log2_T=9,
                                width=width, n_hidden=2, seed=i))
    rays_np = np.resize(adversarial_rays(rng, 16, n_random=300).astype(np.float32), (3001, 8))
    print(f"pairs {feat}/{mlp}: 4 objects x {len(rays_np)} rays", flush=True)
    ctx = L.lsnif_create(0)
    try:
        ids = [L.lsnif_build(ctx, L.ObjectDesc(o, feat, mlp)) for o in objs]
        eye = np.concatenate([np.eye(3), np.zeros((3, 1))], 1).astype(np.float32)
        inst = torch.from_numpy(L.instances_array([(i, eye) for i in ids])).cuda()
        n = len(rays_np)
        rays = torch.from_numpy(np.tile(rays_np, (4, 1))).cuda()
        pr = torch.arange(4 * n, dtype=torch.int32, device="cuda")
        pi = torch.repeat_interleave(torch.arange(4, dtype=torch.int32, device="cuda"), n)
        out = torch.empty((4 * n, 6), dtype=torch.float32, device="cuda")
        L.lsnif_query_pairs(ctx, rays, pr, pi, inst, out)
        one = torch.empty((n, 6), dtype=torch.float32, device="cuda")
        for i, oid in enumerate(ids):
            L.lsnif_query(ctx, oid, rays[:n], one)
            torch.cuda.synchronize()
            got = out[i * n:(i + 1) * n].cpu().numpy()
            want = one.cpu().numpy()
            assert got[:, [0, 1, 5]].tobytes() == want[:, [0, 1, 5]].tobytes(), i   # normals are renormalised
            assert np.allclose(got[:, 2:5], want[:, 2:5], atol=1e-6)
    finally:
        L.lsnif_destroy(ctx)
