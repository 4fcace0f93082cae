"""The launch orders of the NS5 products over a set (host arithmetic): every tile
once, and by a count of its own that no list ends later than the orders it was chosen
from: matrices, or eighths of them, in turn, or balanced by work."""
import ctypes
import heapq

import pytest

import paper_2608_20818_amd as prm

GRAM, POLY, APPLY = 0, 1, 2


def dit(blocks, h):
    return [(h, 3 * h), (h, h), (h, 4 * h), (4 * h, h), (h, 6 * h)] * blocks


def work_list(shapes, factored, kind):
    L = prm.load()
    n, rows, cols = prm._shape_arrays(shapes)
    cfg = prm.config_default()
    k = L.prm_internal_work_list(n, rows, cols, ctypes.byref(cfg), factored, kind, None, 0)
    out = (ctypes.c_int32 * (2 * k))()
    assert L.prm_internal_work_list(n, rows, cols, ctypes.byref(cfg), factored, kind, out, k) == k
    return [(out[2 * i], out[2 * i + 1] >> 16, out[2 * i + 1] & 0xffff) for i in range(k)]


def tile_of(shapes):
    """The planner's tile edge, from the square's tiles of the largest matrix."""
    big = max(range(len(shapes)), key=lambda i: min(shapes[i]))
    f = int(max(shapes[big]) >= 2 * min(shapes[big]))
    t = sum(m == big for m, _, _ in work_list(shapes, f, POLY))
    return next(e for e in (64, 128, 256) if (r := -(-min(shapes[big]) // e)) * (r + 1) // 2 == t)


COST = {256: (1.17, 9.0, 32), 128: (0.42, 5.0, 32), 64: (0.16, 3.5, 96)}


def end(lists, tile):
    stage, fixed, slots = COST[tile]
    last = 0.0
    for ks in lists:
        h = [0.0] * slots
        for k in ks:
            heapq.heappush(h, heapq.heappop(h) + k / 64 * stage + fixed)
        last = max(last, max(h))
    return last


def in_turn(mats, pieces):
    per = [[] for _ in range(8)]
    for i, (n, k) in enumerate(mats):
        for x in range(pieces):
            per[i % 8 if pieces == 1 else x] += [k] * (n * (x + 1) // pieces - n * x // pieces)
    order = [v[j] for j in range(max(map(len, per))) for v in per if j < len(v)]
    return [order[x::8] for x in range(8)]


SETS = {"three blocks of 1280": dit(3, 1280), "three of 1408": dit(3, 1408), "three of 1536": dit(3, 1536),
        "five of 1600": dit(5, 1600), "six of 1024": dit(6, 1024), "three of 2048": dit(3, 2048),
        "four of 3072": dit(4, 3072), "two of 384": dit(2, 384), "one of 1024": dit(1, 1024),
        "tiny": [(256, 256), (256, 256), (256, 768), (256, 1024), (1024, 256), (128, 512)],
        "mixed": [(2938, 5876), (1649, 6596), (900, 2700), (2467, 9000), (1200, 3600), (2201, 2500)] * 2,
        "one": [(2048, 6144)], "small": [(1, 64), (64, 1), (3, 3)]}


@pytest.mark.parametrize("name", sorted(SETS))
def test_every_tile_once(name):
    shapes = SETS[name]
    t = tile_of(shapes)
    for factored in (0, 1):
        for kind in (GRAM, POLY, APPLY):
            want = set()
            for i, s in enumerate(shapes):
                r, c = min(s), max(s)
                if (c >= 2 * r) != bool(factored):
                    continue
                tr, tc = -(-r // t), -(-c // t)
                want |= {(i, a, b) for a in range(tc if kind == APPLY else tr) for b in range(tr)
                         if kind == APPLY or b >= a}
            got = [x for x in work_list(shapes, factored, kind) if x[0] >= 0]
            assert len(got) == len(want) and set(got) == want, (factored, kind)


@pytest.mark.parametrize("name", sorted(SETS))
def test_no_list_ends_later_than_matrices_in_turn(name):
    shapes = SETS[name]
    t = tile_of(shapes)

    def pad(v):
        return -(-v // t) * t

    for factored in (0, 1):
        group = [i for i, s in enumerate(shapes) if (max(s) >= 2 * min(s)) == bool(factored)]
        # the planner's order: by shape padded to 256, largest first
        group.sort(key=lambda i: (-(-min(shapes[i]) // 256), -(-max(shapes[i]) // 256)), reverse=True)
        for kind in (GRAM, POLY, APPLY):
            k = {i: pad((max if kind == GRAM else min)(shapes[i])) for i in group}
            items = work_list(shapes, factored, kind)
            lists = [[k[m] for m, _, _ in items[x::8] if m >= 0] for x in range(8)]
            tiles = {i: sum(m == i for m, _, _ in items) for i in group}
            if not items:
                continue
            turn = end(in_turn([(tiles[i], k[i]) for i in group], 8 if kind == APPLY else 1), t)
            assert end(lists, t) <= 1.031 * turn, (factored, kind)


def test_lists_that_save_no_time_stay_in_turn():
    # one r in a group and no time to save: matrix i of the group on XCD i mod 8, the
    # tiles in their order, no fillers; every XCD an eighth of every matrix of the apply
    for shapes in (dit(3, 1280), dit(3, 1536), dit(5, 1600)):
        assert tile_of(shapes) == 256
        for factored in (0, 1):
            for kind in (POLY, APPLY):
                items = work_list(shapes, factored, kind)
                mats = list(dict.fromkeys(m for m, _, _ in items))
                order = {m: [i for i in items if i[0] == m] for m in mats}
                per = [[] for _ in range(8)]
                if kind == POLY:
                    for j, m in enumerate(sorted(mats, key=lambda m: items.index(order[m][0]))):
                        per[j % 8] += order[m]
                    assert items == [v[j] for j in range(max(map(len, per))) for v in per if j < len(v)]
                else:
                    n = len(order[mats[0]]) // 8
                    assert mats[0] >= 0 and [i[0] for i in items[:8 * n]] == [mats[0]] * (8 * n)


def test_balanced_lists_where_they_save_time():
    # twelve Grams of K = 6144 to 12288, and r x r products of several r
    for shapes, kind in ((dit(3, 2048), GRAM), (SETS["mixed"], POLY)):
        t = tile_of(shapes)
        items = work_list(shapes, 1, kind)
        assert any(m < 0 for m, _, _ in items) or kind == GRAM
        f = max if kind == GRAM else min
        load = [sum(-(-f(shapes[m]) // t) for m, _, _ in items[x::8] if m >= 0) for x in range(8)]
        assert max(load) <= 1.03 * sum(load) / 8


def test_small_tiles_have_room_for_the_fifth_split_matrix():
    # factored form around every tile edge and both sides of its aspect ratio
    cfg = prm.config_default()
    for r in range(1, 700):
        for c in (2 * r, 2 * r + 1, 2 * r + 63, 3 * r):
            assert prm.plan_workspace_bytes([(r, c)], cfg) > 0
