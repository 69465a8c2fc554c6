"""Gradients of the training step's kernel entry by entry: those that rays of at least 8 of 32 parts of the
batch contribute to are held to the per-entry bound of the training tests, 1e-4 of the sum of the
absolute values of the entry's terms.  (An entry of one term says little relative to itself: its
activation may nearly cancel.  With 8 parts the others carry the sum.)"""
import numpy as np
import pytest

import oracle.train as OT
from tests.test_gpu_train import L, gpu_grads, margin_keep, mesh, subset   # noqa: F401
from tests.test_gpu_train_step import SHAPES, shaped
from tests import test_gpu_train_rows as rows
from workloads import train as WT

pytestmark = pytest.mark.gpu

OBJECTS = {**{n: shaped for n in SHAPES}, **{n: rows.shaped for n in rows.SHAPES}}


def held(gpu, ref, ref_abs, parts, what):
    many = parts >= 8
    err, tol = np.abs(gpu.astype(np.float64) - ref)[many], 1e-4 * ref_abs[many]
    print(what, int(many.sum()), "entries held, worst", float((err / tol).max()), flush=True)
    assert np.all(err <= tol), (what, int((err > tol).sum()), float((err / tol).max()))
    return int(many.sum())


@pytest.mark.parametrize("name", sorted(OBJECTS))
def test_entries_of_many_rays(L, mesh, name):   # noqa: F811
    obj = OBJECTS[name](name)
    rays, tg = WT.batch(mesh, obj, 3000, seed=37)
    rays, tg = subset(rays, tg, margin_keep(obj, rays, tg))
    ref = OT.train_grads(obj, rays, tg, bounds=True)
    parts = None
    for part in np.array_split(np.arange(len(rays)), 32):
        g = OT.train_grads(obj, *subset(rays, tg, part), bounds=True)
        hit = [(a > 0).astype(np.int32) for a in [g["gtab_abs"], *g["gW_abs"]]]
        parts = hit if parts is None else [a + b for a, b in zip(parts, hit)]
    loss, gtab, gW, _, _, _ = gpu_grads(L, obj, rays, tg)
    assert abs(loss - ref["loss"]) <= 1e-5 * ref["loss"], (loss, ref["loss"])
    n = held(gtab, ref["gtab"], ref["gtab_abs"], parts[0], f"{name}: tables")
    assert n > 500
    for k in range(len(gW)):
        assert held(gW[k], ref["gW"][k], ref["gW_abs"][k], parts[1 + k], f"{name}: layer {k}") > 100
