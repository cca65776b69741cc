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
