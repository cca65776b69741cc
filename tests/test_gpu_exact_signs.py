"""GPU tests of the 8-slot kernels' exact signs (a whole wavefront evaluates one
lane's table in fp64): exactly degenerate polygons in 8 slots, alone, beside
ordinary pairs, and in wavefronts that the pairs do not fill."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import IOU_TOL, dev_t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as m
    return m


def _pairs(n, every):
    """n pairs in 8 slots: degenerate quadrilaterals (contacts of every kind) at
    each `every`-th place, ordinary 3..8-gons elsewhere."""
    d = synth.c4_polygons(n=n, seed=n)
    a, an, b, bn = (d[k].copy() for k in ("a_xy", "a_nv", "b_xy", "b_nv"))
    qa, qb, _ = synth.degenerate_stress()
    for t, i in enumerate(range(0, n, every)):
        for xy, nv, q in ((a, an, qa), (b, bn, qb)):
            xy[i] = 0.0
            xy[i, :4] = q[t % len(q)]
            nv[i] = 4
    return a, an, b, bn


@pytest.mark.parametrize("every", [1, 7])
@pytest.mark.parametrize("n", [1, 63, 65, 130, 400])
def test_exact_signs_in_8_slots(dg, n, every):
    a, an, b, bn = _pairs(n, every)
    ta, tan, tb, tbn = dev_t(a), dev_t(an), dev_t(b), dev_t(bn)
    ref_iou, ref_nx, ref_xf, bad = oracle.iou_pairs(a, b, an, bn, threads=4)
    assert bad == 0
    iou, nx, xf = (t.cpu().numpy() for t in dg.iou_pairs(ta, tb, tan, tbn))
    assert np.array_equal(nx, ref_nx) and np.array_equal(xf, ref_xf)
    assert np.abs(iou - ref_iou).max() <= IOU_TOL
    xy, nx, xf = (t.cpu().numpy() for t in dg.intersect(ta, tb, tan, tbn))
    assert np.array_equal(nx, ref_nx) and np.array_equal(xf, ref_xf)
    # simple polygons: the crossings are the convex path's crossing codes
    iou, xm, _, _ = (t.cpu().numpy() for t in dg.iou_simple_pairs(ta, tb, tan, tbn))
    want = np.zeros(n, np.uint64)
    for i in range(n):
        for c in ref_xf[i, :ref_nx[i]]:
            if c >= 0x40:
                want[i] |= np.uint64(1) << np.uint64(8 * ((c >> 3) & 7) + (c & 7))
    assert np.array_equal(xm.view(np.uint64), want)
    assert np.abs(iou - ref_iou).max() <= IOU_TOL


@pytest.mark.parametrize("n", [1, 64, 70])
def test_exact_signs_of_matrix_entries(dg, n):
    a, an, b, bn = _pairs(n, 2)
    iou, saved, _ = dg.iou_matrix(dev_t(a), dev_t(b), dev_t(an), dev_t(bn), save=True)
    i, j = (v.ravel() for v in np.meshgrid(np.arange(n), np.arange(n), indexing="ij"))
    ref, nx, xf = oracle.iou_index_pairs(i, j, a, b, an, bn, threads=8)
    assert np.abs(iou.cpu().numpy().ravel() - ref).max() <= IOU_TOL
    cnt = int(saved.count.item())
    pid = saved.pair_id[:cnt].cpu().numpy()
    assert np.array_equal(saved.nx[:cnt].cpu().numpy(), nx[pid])
    assert np.array_equal(saved.xflags[:cnt].cpu().numpy(), xf[pid])
