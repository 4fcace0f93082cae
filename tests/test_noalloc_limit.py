"""Which steps the allocation-free entry point takes: the limit in prm.h, priced
with work lists for 256-wide pieces whatever the kernels' pieces are, at and around
the shapes where the limit lies (host arithmetic), and the bits of a step there."""
import ctypes
import random

import pytest
import torch

import paper_2608_20818_amd as prm

LIMIT = 256 << 20
ITEM, TILE = 16, 256


def a256(x):
    return (x + 255) // 256 * 256


def needed_refresh(m, n, tile=TILE):
    """The same of a refresh step with work lists for tiles of that edge; the
    workspace's padding is to 256 always."""
    r, c = min(m, n), max(m, n)
    rp, cp = -(-r // TILE) * TILE, -(-c // TILE) * TILE
    small = a256(4 * ((rp // 64) * (cp // 64) + 1))
    splits = 4 if c >= 2 * r else 2
    big = 2 * a256(2 * rp * cp) + splits * (a256(2 * rp * rp) + a256(4 * rp))
    T, tc = -(-r // tile), -(-c // tile)
    items = (T * tile // 64) * (tc * tile // 64) + T * (T + 1) // 2 + tc * T
    return 512 + a256(items * ITEM) + a256(small) + big


def needed(m, n):
    """Scratch bytes of a step: 256 for the descriptor, 256 for the int lists, the
    work lists, the prologue's tile sums and alpha, and the workspace."""
    r, c = min(m, n), max(m, n)
    rp, cp = -(-r // TILE) * TILE, -(-c // TILE) * TILE
    small = a256(4 * ((rp // 64) * (cp // 64) + 1))
    if m > n:
        nrb, slabs = -(-m // 32), -(-n // 256)
        items, big = nrb * slabs + slabs, a256((nrb + 1) * n * 4)
    else:
        items, big = 0, 0
    return 512 + a256(max(items, 1) * ITEM) + a256(small) + big


def plan(m, n, refresh):
    L = prm.load()
    L.prm_internal_noalloc_plan.argtypes = [ctypes.POINTER(prm.Config), ctypes.c_int64, ctypes.c_int64, ctypes.c_int64,
                                            ctypes.POINTER(ctypes.c_uint64)]
    out = (ctypes.c_uint64 * 4)()
    rc = L.prm_internal_noalloc_plan(ctypes.byref(prm.config_default(K=2)), m, n, 0 if refresh else 1, out)
    assert rc in (0, 1)
    return rc, list(out)


def largest(f, lo, hi):
    """Largest x in [lo, hi) with f(x) within the limit."""
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if f(mid) <= LIMIT else (lo, mid)
    return lo


@pytest.mark.parametrize("n", [1, 3, 36, 257, 1000, 7616, 23000])
def test_rowwise_steps_of_tall_matrices_up_to_the_limit(n):
    top = largest(lambda m: needed(m, n), n + 1, 1 << 24)
    for m in {n + 1, top - 33, top - 1, top, top + 1, top + 33}:
        if n < m <= 1 << 24:
            ok, (_, _, end, array) = plan(m, n, False)
            assert ok == (needed(m, n) <= LIMIT), (m, n)
            assert not ok or end <= array


def test_a_tall_matrix_just_under_the_limit_is_taken():
    assert needed(275424, 7616) == 268432640
    assert plan(275424, 7616, False)[0] == 1


@pytest.mark.parametrize("r", [1, 64, 200, 256, 512, 700, 1536, 3072, 5000])
def test_refresh_steps_up_to_the_limit(r):
    rng = random.Random(r)
    top = largest(lambda c: needed_refresh(r, c), r, 1 << 24)
    for c in {r, top - 256, top - 1, top, top + 1, top + 300, rng.randint(r, top)}:
        if r <= c <= 1 << 24:
            for m, n in ((r, c), (c, r)):
                ok, (tile, _, end, array) = plan(m, n, True)
                assert tile in (64, 128, 256)
                assert ok == (min(needed_refresh(m, n), needed_refresh(m, n, tile)) <= LIMIT), (m, n)
                assert not ok or end <= array


def test_the_tile_does_not_depend_on_the_limit():
    # 256 x 261120 and 512 x 129792 fit only by the lists of 256-wide tiles; like
    # their neighbours well within the limit they run on 64
    for m, n in ((256, 261120), (512, 129792)):
        assert needed_refresh(m, n) <= LIMIT < needed_refresh(m, n, 64)
        for k in (n, n // 2):
            ok, (tile, _, _, _) = plan(m, k, True)
            assert (ok, tile) == (1, 64)


def same_as_a_context(m, n, t):
    """The step of prm_step_noalloc and of a one-matrix context: the same bits."""
    cfg = prm.config_default(K=2, lr=0.02, wd=0.1)
    gen = torch.Generator(device="cuda").manual_seed(5)
    G = torch.empty(m, n, dtype=torch.bfloat16, device="cuda").normal_(0, 0.01, generator=gen)
    Wa = torch.empty(m, n, dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=gen)
    Ma = torch.empty(m, n, device="cuda").normal_(0, 0.02, generator=gen)
    Wb, Mb = Wa.clone(), Ma.clone()
    print(f"  {m}x{n} t={t}", flush=True)
    with prm.Optimizer([(m, n)], cfg) as opt:
        rho = opt.step([Wa], [G], [Ma], t)
        torch.cuda.synchronize()
    assert prm.step_noalloc(cfg, Wb, G, Mb, t) == rho
    torch.cuda.synchronize()
    assert torch.equal(Ma, Mb) and torch.equal(Wa, Wb)


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_rowwise_step_just_under_the_limit():
    same_as_a_context(275424, 7616, 1)
    torch.cuda.empty_cache()


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
@pytest.mark.parametrize("m,n", [(256, 261120), (129792, 512)])
def test_refresh_step_where_long_lists_pass_the_limit(m, n):
    same_as_a_context(m, n, 0)
