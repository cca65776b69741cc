"""GPU tests of the matrix cull and list passes where they can go wrong: the
masks' bins on spread, coinciding and outlying coordinates against the plain
bounds test, and the output fill on blocks with gaps between them."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_t
from test_gpu_matrix import _check_matrix_exact, _saved_entries

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as m
    return m


def _boxes(rng, n, spread):
    """Boxes 1 x 2 spread over a square of the given side."""
    return synth.boxes_to_quads(rng.uniform(0, spread, n), rng.uniform(0, spread, n),
                                np.full(n, 1.0), np.full(n, 2.0), rng.uniform(-np.pi, np.pi, n))


def _survivors(a, b, az, bz):
    """The bounds test on every pair: closed boxes, open z-extents (empty
    ones meet nothing)."""
    lo, hi, blo, bhi = a.min(1), a.max(1), b.min(1), b.max(1)
    keep = ((lo[:, None] <= bhi[None]) & (blo[None] <= hi[:, None])).all(-1)
    if az is not None:
        keep &= (az[0][:, None] < bz[1][None]) & (bz[0][None] < az[1][:, None])
        keep &= (az[1] > az[0])[:, None] & (bz[1] > bz[0])[None]
    return keep


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("kind", ["spread", "outlier_first", "one_place", "touching", "ragged"])
def test_survivors_are_the_overlapping_bounds(dg, kind, rows):
    rng = np.random.default_rng(len(kind) * 10 + rows)
    na, nb = {"ragged": (65, 1), "spread": (257, 515), "outlier_first": (130, 513),
              "one_place": (300, 129), "touching": (64, 64)}[kind]
    a, b = _boxes(rng, na, 40.0), _boxes(rng, nb, 40.0)
    if kind == "outlier_first":  # the bins' range is taken from these columns
        b[:64] += np.float32(3e4)
        b[70] -= np.float32(1e7)
    if kind == "one_place":  # no extent at all to bin: every column the same box
        b[:] = b[0]
        a[::2] = b[0]
    if kind == "touching":  # a grid of unit squares: closed bounds share sides
        sq = np.array([[0, 0], [1, 0], [1, 1], [0, 1]], np.float32)
        g = np.stack(np.meshgrid(np.arange(8), np.arange(8)), -1).reshape(-1, 1, 2)
        a, b = (sq + g).astype(np.float32), (sq + g[::-1] - 3).astype(np.float32)
    for z in (False, True):
        az = bz = None
        if z:
            az = [rng.integers(0, 6, na).astype(np.float32)]
            bz = [rng.integers(0, 6, nb).astype(np.float32)]
            az.append(az[0] + rng.integers(0, 3, na).astype(np.float32))  # some empty, many touch
            bz.append(bz[0] + rng.integers(0, 3, nb).astype(np.float32))
        t = lambda v: None if v is None else tuple(dev_t(x) for x in v)
        seg = dg.segments(na, nb, None)
        sv = dg.SavedPairs(na * nb, 8, seg[5], torch.device("cuda"), tile_rows=rows)
        _, saved, _ = dg.iou_matrix(dev_t(a), dev_t(b), a_z=t(az), b_z=t(bz), save=True, seg=seg,
                                    saved=sv)
        pid, _, _, _ = _saved_entries(saved)
        want = np.nonzero(_survivors(a, b, az, bz).ravel())[0]
        assert int(saved.count.item()) == len(want)
        assert np.array_equal(np.sort(pid), want), (kind, rows, z)


@pytest.mark.parametrize("nseg,self_pairs,shift", [(5, True, 1), (5, False, 3), (300, True, 2),
                                                   (300, False, 0)])
def test_blocks_with_gaps(dg, nseg, self_pairs, shift):
    """Blocks laid out with gaps, in an output that starts `shift` values past
    a 16-byte boundary: every block's values, and the gaps left alone."""
    rng = np.random.default_rng(nseg + shift)
    na = rng.integers(0, 90 if nseg < 100 else 9, nseg)
    na[1] = 0
    nb = na if self_pairs else rng.integers(0, 70 if nseg < 100 else 9, nseg)
    off = lambda n: np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    a_off, b_off = off(na), off(nb)
    size, gap = na * nb, rng.integers(0, 12, nseg)
    out_off = (off(size + gap)[:-1] + 2).astype(np.int64)
    total = int(out_off[-1] + size[-1] + 7)
    a = _boxes(rng, a_off[-1], 9.0)
    b = a if self_pairs else _boxes(rng, b_off[-1], 9.0)
    ta, tb = dev_t(a), dev_t(a) if self_pairs else dev_t(b)
    if self_pairs:
        tb = ta
    buf = torch.full((total + shift + 4,), -7.0, device="cuda")
    out = buf[shift:shift + total]
    dev = [dev_t(v) for v in (a_off, b_off, out_off)]
    _, _, _, _, _, tiles, _ = dg.segments(len(a), len(b), a_off, b_off, self_pairs=self_pairs)
    sv = dg.SavedPairs(max(1, int(size.sum())), 8, tiles, torch.device("cuda"))
    st = sv.struct()
    pa, pb = dg.polys(ta)[0], dg.polys(tb)[0]
    status = dg.lib.dgal_iou_matrix(dg.context(), pa, pb, *(v.data_ptr() for v in dev), nseg,
                                    int(self_pairs), out.data_ptr(), total, ctypes.byref(st),
                                    torch.cuda.current_stream().cuda_stream)
    assert status == dg.DGAL_OK
    dg.check_errors()
    got = buf.cpu().numpy()[shift:shift + total]
    inside = np.zeros(total, bool)
    for o, n in zip(out_off, size):
        inside[o:o + n] = True
    assert (got[~inside] == -7.0).all() and (buf[:shift] == -7.0).all()
    assert (buf[shift + total:] == -7.0).all()
    _check_matrix_exact(got[inside], a, b, a_off=a_off, b_off=b_off, self_pairs=self_pairs)


@pytest.mark.parametrize("nseg", [1, 7, 4096])
def test_segment_table_forms(dg, nseg):
    """The segment table is the same for offsets given as a list, an array, a
    host tensor of either width or a device tensor (then used as it is), and an
    empty work list is refused."""
    rng = np.random.default_rng(nseg)
    na, nb = rng.integers(0, 600, nseg), rng.integers(0, 600, nseg)
    off = lambda n: np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    a, b = off(na), off(nb)
    size = na * nb
    tiles = {r: int((-(-na // r) * -(-nb // (2048 // r))).sum()) for r in dg.TILE_ROWS_CHOICES}
    for form in (list, np.asarray, torch.tensor, lambda v: torch.tensor(v).int(),
                 lambda v: torch.tensor(v).cuda()):
        fa, fb = form(a), form(b)
        d_a, d_b, d_o, n, total, most, by = dg.segments(int(a[-1]), int(b[-1]), fa, fb)
        assert (n, total, most, by) == (nseg, int(size.sum()), max(tiles.values()), tiles)
        for got, want in ((d_a, a), (d_b, b), (d_o, off(size)[:-1])):
            assert got.is_cuda and got.dtype == torch.int64 and got.is_contiguous()
            assert np.array_equal(got.cpu().numpy(), want)
        if isinstance(fa, torch.Tensor) and fa.is_cuda:
            assert d_a.data_ptr() == fa.data_ptr() and d_b.data_ptr() == fb.data_ptr()
    xy = dev_t(_boxes(rng, 9, 5.0))
    with pytest.raises(dg.DgalError) as e:
        dg.iou_matrix(xy, xy, capacity=0)
    assert e.value.status == dg.DGAL_EINVAL


def test_host_offsets_under_capture(dg):
    """Offsets still on the host are refused under capture (a replay would read
    memory that has been given back), and the table may also stay on the host."""
    rng = np.random.default_rng(3)
    xy = dev_t(_boxes(rng, 40, 5.0))
    off = [0, 15, 40]
    seg = dg.segments(40, 40, off, self_pairs=True)
    saved = dg.SavedPairs(1 << 16, 8, seg[5], xy.device)
    want = dg.iou_matrix(xy, self_pairs=True, seg=seg)[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(RuntimeError):
            dg.iou_matrix(xy, a_off=off, self_pairs=True, check=False, saved=saved)
        with pytest.raises(RuntimeError):
            dg.segments(40, 40, off, self_pairs=True)
        got = dg.iou_matrix(xy, self_pairs=True, check=False, seg=seg, saved=saved)[0]
    for _ in range(3):
        got.zero_()
        graph.replay()
        assert torch.equal(got, want)
        torch.cuda.synchronize()
    host = dg.segments(40, 40, off, self_pairs=True, device="cpu")
    assert [v.tolist() for v in host[:3]] == [off, off, [0, 225]]
