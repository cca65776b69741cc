"""A pair's gradient does not depend on the other pairs of its wavefront, also
where its own vertices are infinite or NaN."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("z3", [False, True])
@pytest.mark.parametrize("side", ["a", "b"])
@pytest.mark.parametrize("kmax,bad", [(8, "inf"), (8, "nan"), (8, "far"), (6, "inf")])
def test_gradient_of_a_pair_alone_and_in_a_batch(kmax, bad, side, z3):
    import paper_2011_11134_amd as dg
    rng = np.random.default_rng(kmax)
    n = 96  # a whole wavefront and half of one
    a, an = synth.workloads.random_convex(rng, n, kmin=kmax, kmax=kmax)
    b, bn = synth.workloads.random_convex(rng, n, kmin=kmax, kmax=kmax)
    special = np.arange(3, n, 5)
    value = {"inf": np.inf, "nan": np.nan, "far": 3e38}[bad]
    # one vertex of one polygon (each in turn), every second pair too far to meet
    (a if side == "a" else b)[special, np.arange(len(special)) % kmax] = value
    a[special[::2]] += np.float32(100.0)
    z = None
    if z3:
        lo = rng.uniform(-1, 0, n).astype(np.float32)
        z = (lo, lo + np.float32(1.5))
    g = rng.uniform(0.5, 1, n).astype(np.float32)
    nx = torch.zeros(n, dtype=torch.uint8, device="cuda")
    xf = torch.full((n, 2 * kmax), 255, dtype=torch.uint8, device="cuda")

    def both(i):
        zz = None if z is None else tuple(dev_t(v[i]) for v in z)
        args = (dev_t(an[i]), dev_t(bn[i]), zz, zz)
        _, nxi, xfi = dg.iou_pairs(dev_t(a[i]), dev_t(b[i]), *args)
        nx[i.tolist()], xf[i.tolist()] = nxi, xfi
        out = dg.iou_pairs_backward(dev_t(a[i]), dev_t(b[i]), dev_t(g[i]), nxi, xfi, *args)
        return [None if t is None else t.cpu().numpy() for t in out]

    batch = both(np.arange(n))
    assert int(nx.max()) > 4  # the batch's other pairs have slots to route
    for i in special:
        for whole, alone in zip(batch, both(np.array([i]))):
            if whole is not None:
                assert np.array_equal(whole[i], alone[0], equal_nan=True), (i, whole[i], alone[0])
    # an empty intersection moves nothing: the finite polygon's gradient is 0
    # (vertex 0 of the first polygon, the origin of the pair's frame, aside)
    empty = special[nx[special.tolist()].cpu().numpy() == 0]
    empty = empty[np.isfinite(a[empty, 0]).all(1)]
    assert not batch[1 if side == "a" else 0][empty].any()
