"""A batch of more than 2^30 rays: the query kernel's work-items, four to a ray, pass the 32 bits that
one launch may have.  The rays are a small batch over and over, and so are the answers."""
import numpy as np
import pytest

from paper_2504_21627_amd import lsnif as L

pytestmark = pytest.mark.gpu


def test_more_rays_than_one_launch():
    import torch
    from tests.test_oracle_pins import tiny_object, adversarial_rays
    torch.cuda.init()
    rng = np.random.default_rng(2)
    obj = tiny_object(8, rng.uniform(size=512) < 0.3, H=2, L=1, F=2, R=[6], log2_T=9, width=64, n_hidden=1, seed=7)
    base = np.resize(adversarial_rays(rng, 8, n_random=400).astype(np.float32), (1024, 8))
    times = (1 << 20) + 3
    n = 1024 * times
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 70 GiB of device memory")
    ctx = L.lsnif_create(0)
    try:
        oid = L.lsnif_build(ctx, L.ObjectDesc(obj, "fp16", "fp16"))
        one = torch.from_numpy(base).cuda()
        want = torch.empty((1024, 6), dtype=torch.float32, device="cuda")
        L.lsnif_query(ctx, oid, one, want)
        rays = one.repeat(times, 1)
        out = torch.full((n, 6), -1.0, dtype=torch.float32, device="cuda")
        print(n, "rays", flush=True)
        L.lsnif_query(ctx, oid, rays, out)
        torch.cuda.synchronize()
        want = want.view(torch.int32)
        assert (want[:, 0] == 1).sum() > 30
        got = out.view(torch.int32).view(times, 1024, 6)
        for a in range(0, times, 1 << 16):
            assert bool((got[a:a + (1 << 16)] == want).all()), a
    finally:
        L.lsnif_destroy(ctx)
        rays = out = got = None
        torch.cuda.empty_cache()
