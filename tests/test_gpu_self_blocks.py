"""Self-pair matrices where their special paths have edges: accepted segments
beside rejected ones."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import dev_t
from test_gpu_matrix import _check_matrix_exact
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
