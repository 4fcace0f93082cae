"""The binding's native tensor checks against its Python ones: what either takes
or refuses, and the pointers they pass on."""
import ctypes
import os

import pytest
import torch

import paper_2608_20818_amd as prm

SHAPES = [(8, 16), (4, 32)]


class Sub(torch.Tensor):
    pass


def test_native_checks_are_built_and_leave_cpu_tensors_to_python():
    assert os.path.exists(os.path.join(os.path.dirname(prm.__file__), "_marshal.so")), "run __graft_entry__.build()"
    from paper_2608_20818_amd import _marshal
    a = (ctypes.c_void_p * 2)()
    spec = _marshal.spec(SHAPES, prm.F32, True)
    for xs in ([torch.zeros(s) for s in SHAPES], [1, 2], [None, None], [torch.zeros(8, 16)], "ab", {}):
        assert _marshal.pointers(spec, xs, ctypes.addressof(a)) is False
    assert list(a) == [None, None]
    with pytest.raises(ValueError):
        _marshal.pointers(object(), [], 0)


def forms(dev):
    """(what it is, a list in place of the gradients)"""
    def good():
        return [torch.ones(s, device=dev) for s in SHAPES]
    g = good()
    yield "plain", g
    yield "tuple", tuple(g)
    yield "parameters", [torch.nn.Parameter(x) for x in g]
    yield "slices", [torch.ones(3, *s, device=dev)[1] for s in SHAPES]
    yield "raw pointers", [x.data_ptr() for x in g]
    yield "a subclass", [x.as_subclass(Sub) for x in g]
    yield "short", g[:1]
    yield "transposed", [g[0].t().contiguous().t(), g[1]]
    yield "wrong shape", [g[0].view(16, 8), g[1]]
    yield "wrong type", [g[0].to(torch.bfloat16), g[1]]
    yield "on the host", [g[0].cpu(), g[1]]
    yield "none", [None, g[1]]
    yield "sparse", [g[0].to_sparse(), g[1]]
    yield "no tensor", ["x", g[1]]


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_native_checks_take_and_refuse_what_the_python_ones_do():
    cfg = prm.config_default(K=2, param_dtype=prm.F32, grad_dtype=prm.F32)
    W = [torch.zeros(s, device="cuda") for s in SHAPES]
    M = [torch.zeros(s, device="cuda") for s in SHAPES]
    with prm.Optimizer(SHAPES, cfg) as opt:
        native = opt._want
        assert all(t._pointers is not None for t in native.values())
        for what, xs in forms("cuda"):
            got = []
            for use in (native, None):
                if use is None:
                    opt._want = {k: prm._Tensors(SHAPES, k, True) for k in native}
                    for t in opt._want.values():
                        t._pointers = None
                else:
                    opt._want = use
                try:
                    got.append([int(v or 0) for v in opt._pointers(xs, prm.F32, "grads")])
                except Exception as e:
                    got.append((type(e), str(e)))
            assert got[0] == got[1], what
            assert isinstance(got[0], list) == (what in ("plain", "tuple", "parameters", "slices", "raw pointers",
                                                         "a subclass")), (what, got)
        opt._want = native

        def under_vmap(g):
            return opt.step(W, [g, g.view(4, 32)], M, 1)

        with pytest.raises(Exception):
            torch.vmap(under_vmap)(torch.ones(2, 8, 16, device="cuda"))
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")
def test_a_configuration_changed_after_construction_is_checked_as_it_stands():
    """A caller may reuse its config object for another context: the storage types it
    then names are held against the tensors, and raw pointers pass."""
    cfg = prm.config_default(K=2, param_dtype=prm.F32, grad_dtype=prm.F32)
    W, G, M = ([torch.zeros(s, device="cuda") for s in SHAPES] for _ in range(3))
    with prm.Optimizer(SHAPES, cfg) as opt:
        cfg.param_dtype = cfg.grad_dtype = prm.BF16
        with pytest.raises(ValueError, match="bfloat16"):
            opt.step(W, G, M, 1)
        assert opt.step(*([x.data_ptr() for x in t] for t in (W, G, M)), 1) == 0
    acfg = prm.adamw_config_default(param_dtype=prm.F32, grad_dtype=prm.F32)
    flat = [torch.zeros(64, device="cuda") for _ in range(4)]
    with prm.AuxAdamW([64], acfg) as aux:
        acfg.param_dtype = prm.BF16
        with pytest.raises(ValueError, match="bfloat16"):
            aux.step(*([x] for x in flat), 1)
        aux.step(*([x.data_ptr()] for x in flat), 1)
    torch.cuda.synchronize()

