"""The row-wise step on rows of any length against the oracle: row lengths on
both sides of every launch class (a wave, a block, the two-sweep path; ragged
ends of 1 to 7 elements), tall matrices on both sides of the separate finalize
and of its rounds, and the one-launch first pass bit for bit against the
separate launches."""
import os
import sys

import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import paper_2608_20818_amd as prm  # noqa: E402
import prm_case as pc  # noqa: E402
from oracle import prm_oracle as po  # noqa: E402

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

SETS = {
    # ragged rows: a wave up to 511, a block of 1 to 8 chunks per thread up to 16391
    "wide": [(3, 7), (5, 9), (2, 511), (6, 513), (3, 2047), (4, 2049), (2, 4097), (3, 6151), (2, 16391), (2, 16393)],
    # aligned ones: a wave up to 4096, a block up to 16384, a larger block up to 32768
    "aligned": [(7, 8), (5, 4096), (3, 4104), (2, 16384), (2, 16392), (1, 32768), (1, 32776)],
    # column widths 1 past and 3 past a multiple of 4; up to 64 row blocks of 32
    # rows (2048) the second pass sums its own norms
    "tall": [(2048, 257), (100, 3), (65, 31), (33, 32), (2047, 260)],
    # beyond: groups of 16 row blocks, a ragged last group, more than one round (64 groups)
    "finalize": [(2049, 257), (16 * 32 * 5 + 1, 36), (16 * 32 * 66 + 40, 5), (700, 100)],
    "mixed": [(9, 513), (513, 9), (40, 520), (520, 40), (64, 64)],
}


@pytest.mark.parametrize("wdt,gdt,nesterov", [(1, 0, 1), (0, 1, 0), (1, 1, 0), (0, 0, 1)])
@pytest.mark.parametrize("name", sorted(SETS))
def test_row_lengths_against_the_oracle(name, wdt, gdt, nesterov):
    shapes = SETS[name]
    cfg = prm.config_default(K=2, lr=0.02, wd=0.1, param_dtype=wdt, grad_dtype=gdt, nesterov=nesterov)
    oc = pc.oracle_config(cfg)
    inputs = pc.host_inputs(shapes, cfg, 87, steps=(1,))
    W = [pc.to_device(w, wdt) for w, _, _ in inputs]
    M = [pc.to_device(m, 0) for _, m, _ in inputs]
    G = [pc.to_device(g[1], gdt) for _, _, g in inputs]
    D = [torch.zeros(s, dtype=torch.float32, device="cuda") for s in shapes]
    W2, M2 = [w.clone() for w in W], [m.clone() for m in M]
    print(f"  {name} W {wdt} G {gdt} nesterov {nesterov}", flush=True)
    with prm.Optimizer(shapes, cfg) as opt:
        assert opt.step(W, G, M, 1, directions=D) == 0
        torch.cuda.synchronize()
        opt.profile_enable(True)  # every launch on its own
        opt.step(W2, G, M2, 1)
        stats = opt.profile_read()
    long_tall = any(m > n and m > 2048 for m, n in shapes)
    assert (stats["rw_tall_finalize"]["launches"] == 1) == long_tall
    for k, (w0, m0, g) in enumerate(inputs):
        Wo, Mo, Do, _ = po.step_matrix(w0, m0, g[1], 1, oc)
        assert pc.rel(pc.to_host(D[k]), Do) <= pc.TOL_ROWWISE, shapes[k]
        assert pc.rel(pc.to_host(M[k]), Mo) <= pc.TOL_M, shapes[k]
        if wdt == prm.BF16:
            assert pc.bf16_write_bound(pc.to_host(W[k]), Wo, pc.to_host(D[k]), Do, cfg.lr) <= 1.0, shapes[k]
        else:  # decay W0 - lr D in fp32: two roundings of each term
            assert pc.rel(pc.to_host(W[k]), Wo) <= 2.0 ** -22, shapes[k]
        assert torch.equal(W[k], W2[k]) and torch.equal(M[k], M2[k]), shapes[k]


@pytest.mark.parametrize("wdt,gdt,nesterov", [(1, 0, 1), (0, 1, 0), (1, 1, 0), (0, 0, 1)])
def test_bits_of_a_matrix_do_not_depend_on_its_set(wdt, gdt, nesterov):
    """Matrices alone and beside so many elements that the launches are split and
    loaded in other ways."""
    few = [(2047, 1001), (65, 31), (700, 100), (9, 513), (64, 64)]
    cfg = prm.config_default(K=2, lr=0.02, wd=0.1, param_dtype=wdt, grad_dtype=gdt, nesterov=nesterov)
    gen = torch.Generator(device="cuda").manual_seed(3)

    def draw(shape, dtype, scale):
        return torch.empty(shape, device="cuda").normal_(0, scale, generator=gen).to(pc.torch_dtype(dtype))

    for more in ([(31000, 2001)], [(2047, 999)] * 12, [(40, 513)] * 300):
        shapes = few + more
        print(f"  W {wdt} G {gdt} nesterov {nesterov} beside {len(more)} of {more[0]}", flush=True)
        W, G, M = ([draw(s, t, x) for s in shapes] for t, x in ((wdt, 0.02), (gdt, 0.01), (0, 0.02)))
        W2, M2 = [w.clone() for w in W[:len(few)]], [m.clone() for m in M[:len(few)]]
        with prm.Optimizer(shapes, cfg) as opt:
            opt.step(W, G, M, 1)
            torch.cuda.synchronize()
        for i, s in enumerate(few):
            with prm.Optimizer([s], cfg) as opt:
                opt.step(W2[i:i + 1], G[i:i + 1], M2[i:i + 1], 1)
                torch.cuda.synchronize()
            assert torch.equal(W[i], W2[i]) and torch.equal(M[i], M2[i]), s
