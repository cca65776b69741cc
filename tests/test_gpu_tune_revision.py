"""Tuned shapes belong to the kernels they were measured on: an entry of
another revision loads and is never taken, and a call that has one shape only
is not tuned."""
import ctypes
import json
import re

import numpy as np
import pytest
import torch

import synth
from gpu_util import dev_t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dg():
    import paper_2011_11134_amd as d
    return d


def _tile_rows(dg, ctx, xy):
    """The tile shape that a forward in the given context takes."""
    n = len(xy)
    pa, _ = dg.polys(xy)
    sv = dg.SavedPairs(n * n, 8, dg.segments(n, n, None)[5], xy.device)
    st = sv.struct()
    out = torch.empty(n * n, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert dg.lib.dgal_iou_matrix(ctx, pa, pa, None, None, None, 0, 0, out.data_ptr(), n * n,
                                  ctypes.byref(st), stream) == dg.DGAL_OK
    assert dg.lib.dgal_check(ctx, stream) == dg.DGAL_OK
    return st.tile_rows


@pytest.mark.parametrize("revision", ["none", "own"])
def test_entries_of_another_revision_are_not_taken(dg, tmp_path, revision):
    rng = np.random.default_rng(2)
    xy = dev_t(synth.boxes_to_quads(*synth.workloads.bev_boxes(rng, 133)))
    dg.set_autotune(True)
    try:
        dg.iou_matrix(xy, xy.clone())
    finally:
        dg.set_autotune(False)
    key = [ln.split(":")[0] for ln in dg.autotune_report()[1].splitlines()
           if "/matrix_fwd" in ln and "seg0" in ln and "/b8.8:" in ln]
    assert len(key) == 1
    key = key[0] if revision == "own" else re.sub(r"(/matrix_fwd)[^/]*/", r"\1/", key[0])
    path = tmp_path / "cache.json"
    path.write_text(json.dumps({"format": "dgal-tune-cache", "version": 1, "entries": [
        {"key": key, "cull_mult": 32, "exact_mult": 4, "tile_rows": 4, "ms": 0.1}]}))
    ctx = ctypes.c_void_p()
    dg.tune_cache_clear()
    try:
        assert dg.tune_cache_load(str(path)) == 1
        assert dg.lib.dgal_create(ctypes.byref(ctx), torch.cuda.current_device()) == dg.DGAL_OK
        assert _tile_rows(dg, ctx, xy) == (4 if revision == "own" else 8)
    finally:
        torch.cuda.synchronize()
        dg.lib.dgal_destroy(ctx)
        dg.tune_cache_clear()


def test_one_shape_is_not_tuned(dg):
    rng = np.random.default_rng(3)
    a, b = (dev_t(synth.boxes_to_quads(*synth.workloads.bev_boxes(rng, n))) for n in (41, 37))
    _, saved, seg = dg.iou_matrix(a, b, save=True)
    g = torch.rand(41 * 37, device="cuda")
    dg.set_autotune(True)
    try:
        dg.iou_matrix_backward(g, saved, seg, a, b)
    finally:
        dg.set_autotune(False)
    assert not [ln for ln in dg.autotune_report()[1].splitlines()
                if "matrix_bwd" in ln and "/b6.6:" in ln]


@pytest.mark.parametrize("n", [1, 300, 70000])
def test_8_slot_backward_on_any_grid(dg, tmp_path, n):
    """The 8-slot pair backward gives the same bits on its resident grid, on one
    workgroup and on a workgroup for every block of pairs."""
    rng = np.random.default_rng(n)
    sets = []
    for _ in range(2):  # 32 polygons, repeated
        xy, nv = synth.workloads.random_convex(rng, 32)
        pick = rng.integers(0, 32, n)
        sets.append((dev_t(xy[pick]), dev_t(nv[pick])))
    (a, an), (b, bn) = sets
    g = torch.rand(n, device="cuda") - 0.5
    _, nx, xf = dg.iou_pairs(a, b, an, bn)
    want = dg.iou_pairs_backward(a, b, g, nx, xf, an, bn)[:2]
    dg.set_autotune(True)
    try:
        dg.iou_pairs_backward(a, b, g, nx, xf, an, bn)
    finally:
        dg.set_autotune(False)
    key = [ln.split(":")[0] for ln in dg.autotune_report()[1].splitlines()
           if "/pairs_bwd" in ln and "/K8/fixed0/z0/" in ln and f"/b{n.bit_length()}:" in ln]
    assert len(key) == 1
    stream = torch.cuda.current_stream().cuda_stream
    for grid in (0, 1, 1 << 24):
        path = tmp_path / f"grid{grid}.json"
        path.write_text(json.dumps({"format": "dgal-tune-cache", "version": 1, "entries": [
            {"key": key[0], "grid": grid, "ms": 0.1}]}))
        ctx = ctypes.c_void_p()
        dg.tune_cache_clear()
        try:
            assert dg.tune_cache_load(str(path)) == 1
            assert dg.lib.dgal_create(ctypes.byref(ctx), torch.cuda.current_device()) == dg.DGAL_OK
            ga, gb = torch.full_like(a, -7.0), torch.full_like(b, -7.0)
            pa, pb = dg.polys(a, an)[0], dg.polys(b, bn)[0]
            assert dg.lib.dgal_iou_backward(ctx, dg.DGAL_PAIRS, pa, pb, None, None, None, 0, 0,
                                            g.data_ptr(), 0, nx.data_ptr(), xf.data_ptr(), None,
                                            ga.data_ptr(), gb.data_ptr(), None, None,
                                            stream) == dg.DGAL_OK
            assert dg.lib.dgal_check(ctx, stream) == dg.DGAL_OK
            assert torch.equal(ga, want[0]) and torch.equal(gb, want[1]), grid
        finally:
            torch.cuda.synchronize()
            dg.lib.dgal_destroy(ctx)
            dg.tune_cache_clear()
