"""GPU tests of row widths: polygon and gradient rows that start off a 16-byte
boundary (8-byte aligned, as the boundary allows) take narrower loads and
stores and give the same bits as aligned ones."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as m
    return m


def _at(t, shift):
    """A copy of t that starts 4 * shift bytes past a 16-byte boundary."""
    buf = torch.full((t.numel() + 8,), -7.0, device="cuda", dtype=torch.float32)
    v = buf[shift:shift + t.numel()].view(t.shape)
    v.copy_(t)
    return v, buf


@pytest.mark.parametrize("kmax", [4, 5, 8])
@pytest.mark.parametrize("n", [1, 127, 300])
def test_simple_rows_off_16_bytes(dg, n, kmax):
    rng = np.random.default_rng(100 * kmax + n)
    ca = rng.uniform(-1, 1, (n, 2))
    a, an = synth.workloads.random_simple(rng, n, ca, kmax=kmax)
    b, bn = synth.workloads.random_simple(rng, n, ca + rng.normal(0, 0.5, (n, 2)), kmax=kmax)
    g = dev_t(rng.uniform(-1, 1, n).astype(np.float32))
    a, an, b, bn = (dev_t(x[:, :kmax] if x.ndim == 3 else x) for x in (a, an, b, bn))
    iou, xm, sm, ins = dg.iou_simple_pairs(a, b, an, bn)
    ga, gb = dg.iou_simple_backward(a, b, g, xm, sm, ins, an, bn)
    for sa, sb, sg in ((2, 0, 0), (0, 2, 0), (0, 0, 2), (2, 2, 2)):
        a2, b2 = _at(a, sa)[0], _at(b, sb)[0]
        iou2, xm2, sm2, ins2 = dg.iou_simple_pairs(a2, b2, an, bn)
        assert torch.equal(iou, iou2) and torch.equal(xm, xm2) and torch.equal(sm, sm2)
        assert torch.equal(ins, ins2)
        ga2, buf_a = _at(torch.zeros_like(ga), sg)
        gb2, buf_b = _at(torch.zeros_like(gb), sg)
        p, q = dg.polys(a2, an)[0], dg.polys(b2, bn)[0]
        st = dg.lib.dgal_iou_simple_backward(
            dg.context(), p, q, g.data_ptr(), xm.data_ptr(), sm.data_ptr(), ins.data_ptr(),
            ga2.data_ptr(), gb2.data_ptr(), torch.cuda.current_stream().cuda_stream)
        assert st == dg.DGAL_OK
        assert torch.equal(ga, ga2) and torch.equal(gb, gb2), (sa, sb, sg)
        for buf in (buf_a, buf_b):  # nothing past the rows
            assert (buf[:sg] == -7).all() and (buf[sg + ga.numel():] == -7).all()


@pytest.mark.parametrize("kmax", [4, 6, 8])
@pytest.mark.parametrize("n", [1, 63, 64, 129, 320])
def test_polygon_rows_off_16_bytes(dg, n, kmax):
    """Intersection polygons and both backwards: whole wavefronts of aligned
    rows go out through LDS, the rest row by row; the bits are the same, and
    nothing is written past the rows."""
    rng = np.random.default_rng(kmax + 10 * n)
    a, an = synth.workloads.random_convex(rng, n, kmax=kmax)
    b, bn = synth.workloads.random_convex(rng, n, kmax=kmax)
    a, an, b, bn = (dev_t(x) for x in (a, an, b, bn))
    g, gx = (dev_t(rng.uniform(-1, 1, s).astype(np.float32)) for s in ((n,), (n, 2 * kmax, 2)))
    pa, pb = dg.polys(a, an)[0], dg.polys(b, bn)[0]
    xy, nx, xf = dg.intersect(a, b, an, bn)
    want = dg.iou_pairs_backward(a, b, g, nx, xf, an, bn)[:2], dg.intersect_backward(
        a, b, gx, nx, xf, an, bn)
    s, ctx = torch.cuda.current_stream().cuda_stream, dg.context()
    for sa, sb in ((0, 2), (2, 0), (2, 2)):
        xy2, buf = _at(torch.zeros_like(xy), sa)
        assert dg.lib.dgal_intersect(ctx, pa, pb, xy2.data_ptr(), nx.data_ptr(), xf.data_ptr(),
                                     s) == dg.DGAL_OK
        assert torch.equal(xy, xy2)
        assert (buf[:sa] == -7).all() and (buf[sa + xy.numel():] == -7).all()
        for k in range(2):
            ga, buf_a = _at(torch.zeros_like(a), sa)
            gb, buf_b = _at(torch.zeros_like(b), sb)
            out = ga.data_ptr(), gb.data_ptr()
            if k == 0:
                st = dg.lib.dgal_iou_backward(ctx, dg.DGAL_PAIRS, pa, pb, None, None, None, 0, 0,
                                              g.data_ptr(), 0, nx.data_ptr(), xf.data_ptr(), None,
                                              *out, None, None, s)
            else:
                st = dg.lib.dgal_intersect_backward(ctx, pa, pb, gx.data_ptr(), nx.data_ptr(),
                                                    xf.data_ptr(), *out, s)
            assert st == dg.DGAL_OK
            assert torch.equal(ga, want[k][0]) and torch.equal(gb, want[k][1]), (sa, sb, k)
            for buf, o, v in ((buf_a, sa, a), (buf_b, sb, b)):
                assert (buf[:o] == -7).all() and (buf[o + v.numel():] == -7).all()
