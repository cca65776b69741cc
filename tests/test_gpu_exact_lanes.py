"""The 8-slot kernels' exact signs around the number of lanes from which each
lane takes its own: 3..8-gons identical to their partners, or sharing a corner,
on a given number of a wavefront's lanes."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import IOU_TOL, dev_t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kmin", [3, 8])
@pytest.mark.parametrize("lanes", [37, 38, 39, 64])
def test_lanes_that_need_exact_signs(lanes, kmin):
    import paper_2011_11134_amd as dg
    rng = np.random.default_rng(lanes + kmin)
    n = 4 * 64 + 41  # the last wavefront is not whole
    w = synth.workloads
    a, an = w.random_convex(rng, n, kmin=kmin)
    b, bn = w.random_convex(rng, n, kmin=kmin)
    for first in range(0, n, 64):
        pick = first + rng.permutation(64)[:lanes]
        for t, i in enumerate(pick[pick < n]):
            if t % 2:  # the same polygon
                b[i], bn[i] = a[i], an[i]
            else:  # moved to share a corner
                b[i, :bn[i]] += a[i, 0] - b[i, 0]
                b[i, 0] = a[i, 0]
    keep = (oracle.simple_status(a, an) == 0) & (oracle.simple_status(b, bn) == 0)
    ta, tan, tb, tbn = dev_t(a), dev_t(an), dev_t(b), dev_t(bn)
    ref, ref_nx, ref_xf, _ = oracle.iou_pairs(a, b, an, bn, threads=4)
    iou, nx, xf = (t.cpu().numpy() for t in dg.iou_pairs(ta, tb, tan, tbn))
    assert np.array_equal(nx[keep], ref_nx[keep]) and np.array_equal(xf[keep], ref_xf[keep])
    assert np.abs(iou - ref)[keep].max() <= IOU_TOL
    _, nx, xf = (t.cpu().numpy() for t in dg.intersect(ta, tb, tan, tbn))
    assert np.array_equal(nx[keep], ref_nx[keep]) and np.array_equal(xf[keep], ref_xf[keep])
    iou, xm, sm, ins = (t.cpu().numpy() for t in dg.iou_simple_pairs(ta, tb, tan, tbn))
    ref, r_xm, r_sm, r_ins, _ = oracle.simple_iou_pairs(a, b, an, bn, threads=4)
    assert np.array_equal(xm.view(np.uint64)[keep], np.asarray(r_xm, np.uint64)[keep])
    assert np.array_equal(sm.view(np.uint64)[keep], np.asarray(r_sm, np.uint64)[keep])
    assert np.array_equal(ins[keep], np.asarray(r_ins, np.uint8)[keep])
    assert np.abs(iou - ref)[keep].max() <= IOU_TOL
    dg.check_errors()
