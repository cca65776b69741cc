"""Survivors of the matrix cull against the plain bounds test on layouts that
take its other paths: words tested whole (far boxes, crowds), bins of ordered
boxes, and both beside the self diagonal."""
import numpy as np
import pytest
import torch

from gpu_util import dev_t
from test_gpu_matrix import _saved_entries
from test_gpu_matrix_cull import _boxes, _survivors

pytestmark = pytest.mark.gpu


def _lay(kind, rng, xy):
    if kind == "sorted":
        return xy[np.argsort(xy[:, 0, 0])]
    if kind == "far_every_64":
        xy[::64] += np.float32(5e4)
    if kind == "far_one_word":  # the other words keep their bins
        xy[70::5] -= np.float32(1e6)
    if kind == "crowd":  # every lane past the one-by-one limit
        xy = (xy * np.float32(0.05)).astype(np.float32)
    if kind == "half_crowd":  # words of both kinds in a wavefront's row
        xy[64:128] *= np.float32(0.02)
        xy[rng.integers(0, len(xy), len(xy) // 3)] *= np.float32(0.02)
    if kind == "infinite":  # bounds without an end, one or both ways
        xy[5, 1, 0] = np.inf
        xy[66, 2, 1] = -np.inf
        xy[129::64, 0] = np.inf
    return xy


KINDS = ["sorted", "far_every_64", "far_one_word", "crowd", "half_crowd", "infinite"]


def _check(dg, rng, kind, rows, na, nb, self_pairs, z, capacity):
    a = _lay(kind, rng, _boxes(rng, na, 40.0))
    b = a if self_pairs else _lay(kind, rng, _boxes(rng, nb, 40.0))
    nb = len(b)
    az = bz = None
    if z:
        heights = lambda n: [rng.uniform(-2, 1, n).astype(np.float32)]
        az = heights(na)
        az.append(az[0] + rng.uniform(-0.2, 2, na).astype(np.float32))  # some empty
        bz = az
        if not self_pairs:
            bz = heights(nb)
            bz.append(bz[0] + rng.uniform(-0.2, 2, nb).astype(np.float32))
    t = lambda v: None if v is None else tuple(dev_t(x) for x in v)
    seg = dg.segments(na, nb, None)
    sv = dg.SavedPairs(capacity, 8, seg[5], torch.device("cuda"), tile_rows=rows)
    more = {"self_pairs": True} if self_pairs else {"b_z": t(bz)}
    _, saved, _ = dg.iou_matrix(dev_t(a), None if self_pairs else dev_t(b), a_z=t(az), save=True,
                                seg=seg, saved=sv, **more)
    pid, _, _, _ = _saved_entries(saved)
    with np.errstate(invalid="ignore"):
        keep = _survivors(a, b, az, bz)
    if self_pairs:
        np.fill_diagonal(keep, False)
    want = np.nonzero(keep.ravel())[0]
    assert len(want) > 0 and int(saved.count.item()) == len(want)
    assert np.array_equal(np.sort(pid), want), (kind, rows, z)


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("self_pairs", [False, True])
def test_survivors(kind, rows, self_pairs):
    import paper_2011_11134_amd as dg
    rng = np.random.default_rng(rows + len(kind))
    for z in (False, True):
        _check(dg, rng, kind, rows, 300, 583, self_pairs, z, 300 * 583)


@pytest.mark.parametrize("rows,kind", [(4, "half_crowd"), (8, "sorted"), (8, "far_every_64"),
                                       (8, "half_crowd"), (16, "infinite")])
@pytest.mark.parametrize("z", [False, True])
def test_survivors_of_a_large_block(kind, rows, z):
    """Past 16.8 M pairs: units of 256 rows, whose last one here is 25 rows."""
    import paper_2011_11134_amd as dg
    rng = np.random.default_rng(rows + len(kind))
    _check(dg, rng, kind, rows, 4121, 4099, False, z, 1 << 23)
