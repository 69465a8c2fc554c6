"""Training steps of objects whose inputs end inside a group of 16 weight rows: with one hidden
layer the head follows the first layer's rows and nothing follows the head; and a weight
that is not finite, on an input that no ray of the batch lists, touches nothing."""
import dataclasses

import numpy as np
import pytest

import oracle
import oracle.train as OT
import workloads as W
from tests.test_gpu_train import L, gpu_grads, margin_keep, mesh, subset   # noqa: F401
from tests.test_gpu_train_step import check_norm
from workloads import train as WT
from workloads.objects import make_object, RELU

pytestmark = pytest.mark.gpu

SHAPES = {   # L, F, H, hidden layers, width, R: inputs
    "8 inputs": (1, 2, 4, 1, 128, [20]),
    "72 inputs": (2, 2, 18, 1, 128, [8, 50]),
    "108 inputs": (2, 3, 18, 1, 128, [64, 100]),
    "42 inputs, width 64": (1, 3, 14, 1, 64, [32]),
    "108 inputs, two layers": (2, 3, 18, 2, 128, [64, 128]),
}


def shaped(name):
    lv, F, H, nh, width, R = SHAPES[name]
    verts, tris = W.icosphere(3)
    return make_object(verts, tris, V=32, bmin=[-1.1] * 3, bmax=[1.1] * 3, L=lv, F=F, log2_T=13, R=R, H=H,
                       n_hidden=nh, width=width, n_mat=4, act=RELU, seed=6, name=name)


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_inputs_that_end_inside_16_rows(L, mesh, name):   # noqa: F811
    obj = shaped(name)
    rays, tg = WT.batch(mesh, obj, 1500, seed=35)
    rays, tg = subset(rays, tg, margin_keep(obj, rays, tg))
    ref = OT.train_grads(obj, rays, tg, bounds=True)
    loss, gtab, gW, _, _, _ = gpu_grads(L, obj, rays, tg)
    print(name, len(rays), loss, ref["loss"], flush=True)
    assert abs(loss - ref["loss"]) <= 1e-5 * ref["loss"], (loss, ref["loss"])
    check_norm(gtab, ref["gtab"], ref["gtab_abs"], "tables")
    for k in range(len(gW)):
        check_norm(gW[k], ref["gW"][k], ref["gW_abs"][k], f"layer {k}")


def test_weights_past_the_listed_points_are_not_used(L, mesh):   # noqa: F811
    """Rays that list at most 2 voxels use the first 24 of 108 inputs: infinite weights on the
    others change no bit of the loss, nor any gradient."""
    obj = shaped("108 inputs, two layers")
    rays, tg = WT.batch(mesh, obj, 6000, seed=36)
    short = oracle.query(obj, rays, debug=True)["count"] <= 4
    rays, tg = subset(rays, tg, short)
    assert len(rays) > 100
    inf = [w.copy() for w in obj.weights]
    inf[0][:, 24:] = np.inf
    want = gpu_grads(L, obj, rays, tg)
    got = gpu_grads(L, dataclasses.replace(obj, weights=inf), rays, tg)
    assert want[0] > 0 and got[0] == want[0]
    for a, b in zip([want[1], *want[2]], [got[1], *got[2]]):
        assert np.isfinite(b).all()
        assert np.abs(a - b).max() <= 1e-5 * np.abs(a).max()   # the tables' atomics are unordered
