"""Matrices where self pairs and the backward's split of the work have edges:
accepted segments beside rejected ones, one block without offsets, and blocks of
more row groups than are resident at once."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import IOU_TOL, dev_t
from test_gpu_matrix import (_aabb_candidates, _assert_box_grads, _box_grads, _check_matrix_exact,
                             _crowd, _grad_reference)
from test_gpu_matrix_cull import _boxes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as m
    return m


@pytest.mark.parametrize("offs,bad", [
    ([0, 50, 20, 40], [1]),              # rows 20..39 belong to both accepted segments
    ([0, 10, 90, 30, 70], [1, 2]),       # past the boxes, then back
    ([5, 70, 60, 64, 64, 80], [1]),
])
def test_accepted_segments_beside_rejected_ones(dg, offs, bad):
    """Every accepted block is written whole (the diagonal exactly 1), a
    rejected one is left alone and reported."""
    rng = np.random.default_rng(len(offs))
    n, nseg = 80, len(offs) - 1
    a = _boxes(rng, n, 9.0)
    off = np.array(offs, np.int64)
    cnt = off[1:] - off[:-1]
    out_off = np.concatenate([[0], np.cumsum(cnt * cnt)]).astype(np.int64)
    total = int(out_off[-1])
    ta = dev_t(a)
    dev = [dev_t(v) for v in (off, out_off[:-1])]
    out = torch.full((total,), -7.0, device="cuda")
    sv = dg.SavedPairs(total, 8, 4096, torch.device("cuda"))
    st = sv.struct()
    pa = dg.polys(ta)[0]
    stream = torch.cuda.current_stream().cuda_stream
    rc = dg.lib.dgal_iou_matrix(dg.context(), pa, pa, dev[0].data_ptr(), dev[0].data_ptr(),
                                dev[1].data_ptr(), nseg, 1, out.data_ptr(), total,
                                ctypes.byref(st), stream)
    assert rc == dg.DGAL_OK
    assert dg.lib.dgal_check(dg.context(), stream) == dg.DGAL_EINVAL
    got = out.cpu().numpy()
    for s in range(nseg):
        block = got[out_off[s]:out_off[s + 1]]
        if s in bad:
            assert (block == -7.0).all(), s
        elif cnt[s]:
            block = block.reshape(cnt[s], cnt[s])
            assert (np.diagonal(block) == 1.0).all(), (s, np.nonzero(np.diagonal(block) != 1.0))
            _check_matrix_exact(block.ravel(), a[off[s]:off[s + 1]], a[off[s]:off[s + 1]],
                                self_pairs=True)


@pytest.mark.parametrize("z3", [False, True])
@pytest.mark.parametrize("n,kmax,factor", [
    (1, 4, 1.0), (7, 4, 0.1), (9, 4, 0.1), (700, 4, 0.1), (1, 8, 1.0), (9, 8, 1.0), (331, 8, 1.0),
    (8209, 4, 1.0),  # more row groups than are resident at once
])
def test_one_self_block(dg, n, kmax, factor, z3):
    """Self pairs of one block without offsets: IoU and its gradient against the
    oracle, the diagonal exactly 1 (700 boxes in a crowd: groups of many steps)."""
    rng = np.random.default_rng(n + kmax)
    an = None
    if kmax == 4:
        w = synth.workloads
        a = _crowd(w.boxes_to_quads(*w.bev_boxes(rng, n)), factor)
    else:
        a, an = synth.workloads.random_convex(rng, n, kmax=kmax, min_turn=0.02)
    z = None
    if z3:
        lo = rng.uniform(-2, 1, n).astype(np.float32)
        z = (lo, (lo + rng.uniform(0.5, 2, n)).astype(np.float32))
    g = rng.uniform(-1, 1, n * n).astype(np.float32)
    tz = None if z is None else tuple(dev_t(v) for v in z)
    ta, tn = dev_t(a), dev_t(an)
    iou, saved, seg = dg.iou_matrix(ta, a_nv=tn, a_z=tz, self_pairs=True, save=True)
    got = iou.cpu().numpy()
    assert got.shape == (n, n) and (np.diagonal(got) == 1.0).all()
    ga, gb, gaz, gbz = dg.iou_matrix_backward(dev_t(g), saved, seg, ta, a_nv=tn, a_z=tz,
                                              self_pairs=True)
    assert gb is None and gbz is None
    dg.check_errors()
    ia, ib, fl = _aabb_candidates(a, a)
    lo_i, hi_i = np.minimum(ia, ib), np.maximum(ia, ib)
    ref, _, _ = oracle.iou_index_pairs(lo_i, hi_i, a, a, an, an, a_z=z, b_z=z, threads=8)
    ref = np.where(ia == ib, 1.0, ref)
    flat = got.ravel()
    assert np.abs(flat[fl].astype(np.float64) - ref).max() <= IOU_TOL
    rest = np.ones(n * n, bool)
    rest[fl] = False
    assert not flat[rest].any()
    if n > 1:
        (ref_g, scale), = [_grad_reference(a, a, g, ia, ib, fl, an, an, z, z, self_pairs=True)]
        _assert_box_grads(_box_grads(ga, gaz), ref_g, scale, "self")
    else:
        assert not ga.any()


@pytest.mark.parametrize("n,m,factor", [
    (8209, 300, 0.2),   # a wavefront a row group, groups of several steps
    (8209, 2048, 1.0),  # a workgroup a row group, more of them than are resident
])
def test_many_row_groups(dg, n, m, factor):
    rng = np.random.default_rng(m)
    w = synth.workloads
    a, b = (_crowd(w.boxes_to_quads(*w.bev_boxes(rng, k)), factor) for k in (n, m))
    g = rng.uniform(-1, 1, n * m).astype(np.float32)
    ta, tb = dev_t(a), dev_t(b)
    _, saved, seg = dg.iou_matrix(ta, tb, save=True)
    ga, gb, _, _ = dg.iou_matrix_backward(dev_t(g), saved, seg, ta, tb)
    dg.check_errors()
    assert factor == 1.0 or int(saved.count.item()) * 8 > 64 * n  # above a step a group on average
    ia, ib, fl = _aabb_candidates(a, b)
    ra, sa, rb, sb = _grad_reference(a, b, g, ia, ib, fl)
    _assert_box_grads(_box_grads(ga), ra, sa, "rows")
    _assert_box_grads(_box_grads(gb), rb, sb, "columns")
