"""The order in which the NS5 input norm is summed: 256 threads, each over the
64 x 64 tile sums t, t + 256, ... one after the other.  alpha = 1 / (norm + eps)
scales every element of the iterate, so another order moves the outputs of a
refresh by a rounding of alpha.

The momentum here has tile sums of 2^24 in the first 256 tiles and of 1 in all the
others: in that order every 1 is absorbed (2^24 + 1 rounds to 2^24), the total is
2^32 and alpha exactly 2^-16.  With b = c = 0 the five iterations multiply by a,
which is chosen so that a times a momentum element is a tie between two bf16
values: an alpha that is one unit smaller rounds the other way, by 2^-7 of the
direction."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import paper_2608_20818_amd as prm  # noqa: E402

TILES = 256 * 64
A = 1 + 3 * 2.0 ** -8


def total(threads):
    """The sum of squares with that many threads, in fp32 (numpy)."""
    p = np.ones(TILES, np.float32)
    p[:256] = 2.0 ** 24
    s = np.zeros(threads, np.float32)
    for row in p.reshape(-1, threads):
        s = s + row
    waves = s.reshape(-1, 64)
    while waves.shape[1] > 1:  # a wave's butterfly: powers of two here, exact in any order
        waves = waves[:, ::2] + waves[:, 1::2]
    t = np.float32(0)
    for w in waves[:, 0]:
        t = np.float32(t + w)
    return t


def test_the_input_tells_the_orders_apart():
    assert total(256) == np.float32(2.0 ** 32)
    assert np.float32(1) / np.sqrt(total(1024), dtype=np.float32) < np.float32(2.0 ** -16)


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_order_of_the_input_norm():
    n = 64 * TILES
    G = torch.zeros(1, n, device="cuda")
    G[0, :256 * 64] = 512.0                # 64 elements of a tile: 2^24
    G[0, 256 * 64::64] = 1.0
    W, M, D = (torch.zeros(1, n, device="cuda") for _ in range(3))
    cfg = prm.config_default(K=1, beta=0.0, lr=1.0, wd=0.0, param_dtype=prm.F32, grad_dtype=prm.F32, ns_plain=1,
                             ns_a=A, ns_b=0.0, ns_c=0.0, eps_ns=1e-12)
    with prm.Optimizer([(1, n)], cfg) as opt:
        assert opt.step([W], [G], [M], 0, directions=[D]) == 1
    torch.cuda.synchronize()
    want = G.cpu() * 2.0 ** -16            # exact
    for _ in range(5):
        want = (want * A).to(torch.bfloat16).float()  # exact product, one rounding
    assert torch.equal(D.cpu(), want)
    assert torch.equal(W.cpu(), -want)
