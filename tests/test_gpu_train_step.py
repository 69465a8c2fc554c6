"""The training step's kernel at the edges of its tiles (32 rays), of its register blocks (20
and 36 32 x 32 blocks of weight gradient, more: the separate products) and of its ray order
(2^18 rays), against the training oracle.

An entry's error is held against the layer's (or the tables') largest entry, 1e-5 of it, the
relative accuracy of the float32 forward and backward values: an entry of few rays, or of a
unit that one ray activates, can be one term whose activation nearly cancels, and says
nothing relative to itself."""
import numpy as np
import pytest

import oracle.train as OT
import workloads as W
from tests.test_gpu_train import L, check_grad, gpu_grads, margin_keep, mesh, subset   # noqa: F401
from workloads import train as WT
from workloads.objects import make_object, LEAKY_RELU, RELU

pytestmark = pytest.mark.gpu

SHAPES = {   # L, F, H, hidden layers, width, R, activation
    "10 blocks": (2, 3, 10, 2, 64, [64, 128], LEAKY_RELU),
    "one hidden layer": (2, 3, 16, 1, 64, [20, 48], RELU),
    "36 blocks": (2, 3, 18, 2, 128, [64, 100], LEAKY_RELU),
    "odd inputs": (3, 2, 14, 2, 128, [8, 32, 77], RELU),
    "more blocks": (1, 3, 14, 3, 128, [96], LEAKY_RELU),
    "many more blocks": (2, 3, 18, 3, 128, [64, 128], LEAKY_RELU),
}


def check_norm(gpu, ref, ref_abs, what):
    err, tol = float(np.abs(gpu.astype(np.float64) - ref).max()), 1e-5 * float(ref_abs.max())
    assert err <= tol, (what, err, tol)


def shaped(name):
    lv, F, H, nh, width, R, act = SHAPES[name]
    verts, tris = W.icosphere(3)
    return make_object(verts, tris, V=32, bmin=[-1.1] * 3, bmax=[1.1] * 3, L=lv, F=F, log2_T=13, R=R, H=H,
                       n_hidden=nh, width=width, n_mat=4, has_albedo=1, act=act, leaky_slope=0.01, seed=5, name=name)


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_step_at_tile_edges(L, mesh, name):   # noqa: F811
    obj = shaped(name)
    rays, tg = WT.batch(mesh, obj, 1500, seed=31)
    rays, tg = subset(rays, tg, margin_keep(obj, rays, tg))
    for n in (1, 31, 33, len(rays)):
        r, t = subset(rays, tg, np.arange(len(rays) - n, len(rays)))
        ref = OT.train_grads(obj, r, t, bounds=True)
        loss, gtab, gW, _, _, _ = gpu_grads(L, obj, r, t)
        print(name, n, loss, ref["loss"], flush=True)
        assert abs(loss - ref["loss"]) <= 1e-5 * ref["loss"], (n, loss, ref["loss"])
        check_norm(gtab, ref["gtab"], ref["gtab_abs"], f"tables, {n} rays")
        for k in range(len(gW)):
            check_norm(gW[k], ref["gW"][k], ref["gW_abs"][k], f"layer {k}, {n} rays")


@pytest.mark.parametrize("which", ["paper", "c1"])
def test_step_of_more_rays_than_two_launches_order(L, mesh, which):   # noqa: F811
    """A batch given many times over has its own mean loss and gradients (c1: 288 inputs, which
    only large batches bring to the one kernel)."""
    obj = W.configs.paper_object(seed=11) if which == "paper" else W.configs.c1_object(seed=2)
    rays, tg = WT.batch(mesh, obj, 2000, seed=33)
    rays, tg = subset(rays, tg, margin_keep(obj, rays, tg))
    ref = OT.train_grads(obj, rays, tg, bounds=True)
    times = (1 << 18) // len(rays) + 1
    many = np.tile(np.arange(len(rays)), times)
    r, t = subset(rays, tg, many)
    assert len(r) > 1 << 18
    loss, gtab, gW, _, _, _ = gpu_grads(L, obj, r, t)
    assert abs(loss - ref["loss"]) <= 1e-5 * ref["loss"], (loss, ref["loss"])
    check = check_grad if which == "paper" else check_norm
    check(gtab, ref["gtab"], ref["gtab_abs"], "tables")
    for k in range(len(gW)):
        check(gW[k], ref["gW"][k], ref["gW_abs"][k], f"layer {k}")
