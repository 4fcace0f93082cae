"""How a row-wise step is launched over a set (host arithmetic): which sets sum the
column norms of tall matrices in the second pass and which in a launch between."""
import ctypes

import pytest

import paper_2608_20818_amd as prm


def plan(shapes, wdt=prm.BF16, gdt=prm.BF16):
    L = prm.load()
    n, rows, cols = prm._shape_arrays(shapes)
    out = (ctypes.c_int32 * 2)()
    cfg = prm.config_default(param_dtype=wdt, grad_dtype=gdt)
    assert L.prm_internal_rowwise_plan(n, rows, cols, ctypes.byref(cfg), out) == prm.PRM_OK
    return list(out)


@pytest.mark.parametrize("shapes,own", [
    ([(1024, 256)] * 3, 1), ([(2048, 512)], 1), ([(2048, 1024)] * 4, 1), ([(1024, 1000)] * 16, 1),
    # beyond 64 row blocks, and beyond what the tiles can read at their start
    ([(2049, 512)], 0), ([(2048, 512)] * 16, 0), ([(2048, 512)] * 64, 0), ([(2047, 1001)] * 16, 0),
    ([(1536, 384)] * 64, 0), ([(256, 256)], 1), ([(64, 128)] * 5, 1), ([], 1)])
def test_own_norms(shapes, own):
    assert plan(shapes)[0] == own


def dit(blocks, h):
    return [(h, 3 * h), (h, h), (h, 4 * h), (4 * h, h), (h, 6 * h)] * blocks


@pytest.mark.parametrize("shapes,first", [
    # long rows, and few blocks: the launches' ends count
    (dit(2, 384), 1), (dit(6, 1024), 1), (dit(3, 2048), 1), ([(9, 513), (513, 9), (64, 64)], 1),
    # many short rows or narrow tiles: two blocks on a CU are too few
    ([(64, 64)] * 200 + [(512, 513)] * 100, 0), ([(3000, 600), (64, 4000)] * 20 + [(500, 520)] * 60, 0),
    # one class, none, and too large
    ([(512, 513)] * 100, 0), ([], 0), (dit(6, 2048), 0)])
def test_one_first_launch(shapes, first):
    assert plan(shapes)[1] == first
