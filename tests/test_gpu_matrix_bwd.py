"""Backward of two-set IoU matrices against the FP64 oracle, where its split of
the work has edges: row groups of 8, steps of 64 entries, the rows of the
second set whose gradients an instruction's atomic adds take together."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_t
from test_gpu_matrix import (_aabb_candidates, _assert_box_grads, _box_grads, _crowd,
                             _grad_reference)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as d
    assert torch.cuda.is_available()
    return d


def _set(rng, n, kmax):
    if kmax == 4:
        w = synth.workloads
        return _crowd(w.boxes_to_quads(*w.bev_boxes(rng, n)), 0.1), None
    return synth.workloads.random_convex(rng, n, kmax=kmax, min_turn=0.02)


def _heights(rng, n):
    lo = rng.uniform(-2, 1, n).astype(np.float32)
    return lo, (lo + rng.uniform(0.5, 2, n)).astype(np.float32)


@pytest.mark.parametrize("z3", [False, True])
@pytest.mark.parametrize("kmax", [4, 6, 8])
@pytest.mark.parametrize("n,m", [(1, 1), (1, 700), (7, 333), (8, 64), (9, 1500), (1031, 9),
                                 (8209, 3)])
def test_two_set_backward(dg, n, m, kmax, z3):
    rng = np.random.default_rng(n + m + kmax)
    (a, an), (b, bn) = _set(rng, n, kmax), _set(rng, m, kmax)
    az, bz = (_heights(rng, n), _heights(rng, m)) if z3 else (None, None)
    g = rng.uniform(-1, 1, n * m).astype(np.float32)
    dev = lambda v: None if v is None else dev_t(v)
    args = [dev(a), dev(b), dev(an), dev(bn)] + [
        None if z is None else tuple(dev(t) for t in z) for z in (az, bz)]
    print(f"case: {n} x {m}, kmax {kmax}, z3 {z3}", flush=True)
    _, saved, seg = dg.iou_matrix(*args, save=True)
    ga, gb, gaz, gbz = dg.iou_matrix_backward(dev(g), saved, seg, *args)
    dg.check_errors()
    ia, ib, fl = _aabb_candidates(a, b)
    ra, sa, rb, sb = _grad_reference(a, b, g, ia, ib, fl, an, bn, az, bz)
    _assert_box_grads(_box_grads(ga, gaz), ra, sa, "rows")
    _assert_box_grads(_box_grads(gb, gbz), rb, sb, "columns")
