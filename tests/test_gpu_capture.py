"""Residual evaluations under stream capture.  An evaluation only launches kernels: it can be captured as the first thing
after any call that changes how it runs (precision, reorder traversal, tuning, moved integrals), and a captured graph
stays valid while precision and traversal change and change back.  Each replay, with eager evaluations between, has to
give the bits of the eager evaluation in the same setting (a setting fixes every order of summation)."""
import numpy as np
import pytest

import fsgen

pytestmark = pytest.mark.gpu


def _setup(real=False, size=(9, 37, 5)):
    import torch
    import paper_2004_03682_amd as F
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    s = fsgen.make_system(*size, 0.05, 17, real=real)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = F.Context.from_system(s, stream=st, precision="real_fp64" if real else "fp64")
        for C in fsgen.CLASSES:
            buf, _ = fsgen.class_buffer(s, C)
            ctx.set_integrals(C, torch.from_numpy(fsgen.real_buffer(buf) if real else buf).cuda())
        rng = np.random.default_rng(4)
        t = [0.02 * (rng.normal(size=n) + 1j * rng.normal(size=n)) for n in (ctx.n1, ctx.n2)]
        t = [torch.from_numpy(x.real.copy() if real else x).cuda() for x in t]
        r = [torch.empty_like(x) for x in t]
    st.synchronize()
    return ctx, st, t, r


def _capture(ctx, st, t, r):
    import torch
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
        ctx.build_residual(*t, *r)
    return g


def _run(st, r, f):
    import torch
    with torch.cuda.stream(st):
        for x in r:
            x.fill_(7.0)
        f()
    st.synchronize()
    return [x.clone() for x in r]


def _out_and_back(ctx):
    ctx.vvvv_out_of_core(1 << 20)
    ctx.vvvv_out_of_core(0)


SETTINGS = {
    "fresh": lambda c: None,
    "storage order": lambda c: c.gather_order(0),
    "affine tiles": lambda c: c.gather_order(2),
    "tuned": lambda c: c.autotune(1),
    "defaults": lambda c: c.autotune(0),
    "integrals moved": _out_and_back,
    "split bf16": lambda c: c.set_precision("split_bf16"),
    "split bf16 and back": lambda c: (c.set_precision("split_bf16"), c.set_precision("fp64")),
}


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("name", list(SETTINGS))
def test_captured_first_thing_after_a_setting(name, real):
    import torch
    if real and name.startswith("split"):
        pytest.skip("a real context computes in FP64 only")
    ctx, st, t, r = _setup(real)
    SETTINGS[name](ctx)
    g = _capture(ctx, st, t, r)
    first = _run(st, r, g.replay)
    for _ in range(3):
        eager = _run(st, r, lambda: ctx.build_residual(*t, *r))
        again = _run(st, r, g.replay)
        for a, b, c in zip(first, eager, again):
            assert torch.equal(a, b) and torch.equal(a, c)
    ctx.destroy()


def test_a_captured_graph_outlives_changes_of_precision_and_traversal():
    import torch
    ctx, st, t, r = _setup()
    g = _capture(ctx, st, t, r)
    first = _run(st, r, g.replay)
    for change in (lambda: ctx.gather_order(2), lambda: ctx.gather_order(0), lambda: ctx.set_precision("split_bf16"),
                   lambda: ctx.gather_order(1), lambda: ctx.set_precision("fp64"), lambda: ctx.gather_order(0)):
        change()
        _run(st, r, lambda: ctx.build_residual(*t, *r))
        again = _run(st, r, g.replay)
        for a, b in zip(first, again):
            assert torch.equal(a, b)
    ctx.destroy()


def _launches(ctx, st, t, r):
    """Kernel launches of one evaluation (nodes of its captured graph)."""
    import ctypes
    import torch
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
        ctx.build_residual(*t, *r)
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    n = ctypes.c_size_t()
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("nocc,nvirt,nirrep", [(9, 37, 5), (14, 86, 1)])
@pytest.mark.parametrize("real", [False, True])
def test_tuning_and_storage_order_replace_a_forced_traversal(nocc, nvirt, nirrep, real):
    """Tuning chooses the traversals anew and level 0 restores those of a fresh context; storage order lets every reorder
    into chains again, also one that tuning had put on tiles (the second system has reorders above 2^19 elements)."""
    ctx, st, t, r = _setup(real, (nocc, nvirt, nirrep))
    fresh = _launches(ctx, st, t, r)
    ctx.gather_order(2)
    forced = _launches(ctx, st, t, r)
    assert forced > fresh
    ctx.autotune(0)
    assert _launches(ctx, st, t, r) == fresh
    ctx.gather_order(2)
    ctx.autotune(1)
    assert _launches(ctx, st, t, r) < forced
    ctx.autotune(0)
    ctx.gather_order(0)
    assert _launches(ctx, st, t, r) == fresh
    ctx.destroy()
