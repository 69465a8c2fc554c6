"""The walk with several lanes per ray (small launches) against the walk with one lane per
ray: the same voxel lists, shown by the encodings and raw outputs they lead to, bit for bit,
at batch sizes on each side of every switch, and the oracle's point counts."""

import dataclasses

import numpy as np
import pytest

import oracle
from paper_2504_21627_amd import lsnif as L

pytestmark = pytest.mark.gpu


def encodings(ctx, oid, obj, rays):
    import torch
    n = len(rays)
    r = torch.from_numpy(np.ascontiguousarray(rays, np.float32)).cuda()
    out = torch.empty((n, 6), dtype=torch.float32, device="cuda")
    bufs = {"enc": torch.zeros((n, obj.H * obj.L * obj.F), dtype=torch.float32, device="cuda"),
            "out": torch.zeros((n, obj.out_dim), dtype=torch.float32, device="cuda"),
            "count": torch.zeros(n, dtype=torch.int32, device="cuda")}
    L.lsnif_query_debug(ctx, oid, r, out, bufs)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in bufs.items()}


# densities: lists that reach the cap, lists that cross long empty stretches
@pytest.mark.parametrize("V,density", [(2, 0.7), (4, 0.5), (32, 0.9), (32, 0.02), (128, 0.3), (128, 0.004), (256, 0.01), (512, 0.002)])
@pytest.mark.parametrize("recheck", [0, 1])
def test_lists_equal_the_serial_walk(V, density, recheck):
    from tests.test_oracle_pins import tiny_object, adversarial_rays, edge_grazing_rays
    rng = np.random.default_rng(V + recheck)
    occ = rng.uniform(size=V ** 3) < density
    obj = tiny_object(V, occ, H=18, L=1, F=2, R=[V], log2_T=10, width=64, n_hidden=1, seed=V)
    obj = dataclasses.replace(obj, grazing_recheck=recheck)
    edge = edge_grazing_rays(rng, V, 300)   # in voxel units of a [0, V] box
    edge = edge.copy()
    edge[:, 0:3] = edge[:, 0:3] * (2.0 / V) - 1.0
    edge[:, 3:6] *= 2.0 / V
    base = np.concatenate([adversarial_rays(rng, V, n_random=400), edge]).astype(np.float32)
    print(f"walk V={V} density={density} recheck={recheck}: {len(base)} rays", flush=True)
    import torch
    torch.cuda.init()
    ctx = L.lsnif_create(0)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(obj, "fp32", "fp32"))
        # one lane per ray: past the last switch
        serial = encodings(ctx, oid, obj, np.resize(base, (57344 + 257, 8)))
        assert np.array_equal(serial["count"][:len(base)], oracle.query(obj, base, debug=True)["count"])
        for n in (1, 63, len(base), 8192, 8193, 32769, 57344):
            got = encodings(ctx, oid, obj, np.resize(base, (n, 8)))
            for k, v in got.items():
                assert v.tobytes() == serial[k][:n].tobytes(), (n, k)
    finally:
        L.lsnif_destroy(ctx)
