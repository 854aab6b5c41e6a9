"""Fused launches of small operations (k_fused): residuals against the dense oracle at sizes around the 16 x 16 tiles,
the 256-element chunks and the K split over waves and workgroups (K = o v^2 / 2 up to 4.5 k here), in complex and
real arithmetic; and against the same operations on kernels of their own (profiling puts every operation there).
Both sums have at most a few thousand terms of size <= max|R|, so 1e-12 of max|R| is asked, as in the parity tests."""
import numpy as np
import pytest

import fsgen
import layout_ref as LR
from oracle import ccsd

pytestmark = pytest.mark.gpu


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _random_t(s, rng, real):
    no, nv = s.nocc, s.nvirt
    go, gv = s.irrep[:no], s.irrep[no:]
    t1 = 0.05 * (rng.normal(size=(no, nv)) + 1j * rng.normal(size=(no, nv)))
    t2 = 0.05 * (rng.normal(size=(no, no, nv, nv)) + 1j * rng.normal(size=(no, no, nv, nv)))
    t2 = t2 - t2.transpose(1, 0, 2, 3)
    t2 = t2 - t2.transpose(0, 1, 3, 2)
    t1 *= go[:, None] == gv[None, :]
    t2 *= ((go[:, None, None, None] + go[None, :, None, None] - gv[None, None, :, None] - gv[None, None, None, :])
           % s.nirrep == 0)
    return (t1.real + 0j, t2.real + 0j) if real else (t1, t2)


@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("nocc,nvirt,nirrep", [(2, 3, 1), (3, 15, 1), (4, 16, 1), (5, 17, 1), (6, 33, 2), (9, 32, 1),
                                               (8, 37, 3), (12, 26, 5)])
def test_fused_residual_matches_oracle_and_single_kernels(nocc, nvirt, nirrep, real):
    import torch
    import paper_2004_03682_amd as F
    s = fsgen.make_system(nocc, nvirt, nirrep, 0.05, 91, real=real)
    ctx = F.Context.from_system(s, precision="real_fp64" if real else "fp64")
    for C in fsgen.CLASSES:
        buf, _ = fsgen.class_buffer(s, C)
        ctx.set_integrals(C, _dev(fsgen.real_buffer(buf) if real else buf))
    t1, t2 = _random_t(s, np.random.default_rng(nvirt), real)
    p1, p2 = LR.pack_t1(s, t1), LR.pack_t2(s, t2)
    if real:
        p1, p2 = p1.real, p2.real
    d1, d2 = _dev(p1), _dev(p2)
    runs = []
    for prof in (False, True):
        ctx.profile(prof)
        r1, r2 = torch.full_like(d1, 3.0), torch.full_like(d2, 3.0)
        ctx.build_residual(d1, d2, r1, r2)
        runs.append((r1.cpu().numpy(), r2.cpu().numpy()))
    R1, R2 = ccsd.residual(ccsd.Dense(s), t1, t2)
    scale = max(np.abs(R1).max(), np.abs(R2).max())
    ref = LR.pack_t1(s, R1), LR.pack_t2(s, R2)
    for r in runs:
        for a, b in zip(r, ref):
            assert a.size == 0 or np.abs(a - b).max() <= 1e-12 * scale
    ctx.destroy()


@pytest.mark.parametrize("real", [False, True])
def test_parts_of_a_tile_meet_in_order_on_every_pass(real):
    """Tiles split over workgroups (K = 2.3 k and 4.6 k): the counters of arrived parts are clear again after each pass,
    and the parts are added in order whoever comes last, so every pass gives the same bits."""
    import torch
    import paper_2004_03682_amd as F
    s = fsgen.make_system(8, 34, 1, 0.05, 92, real=real)
    ctx = F.Context.from_system(s, precision="real_fp64" if real else "fp64")
    for C in fsgen.CLASSES:
        buf, _ = fsgen.class_buffer(s, C)
        ctx.set_integrals(C, _dev(fsgen.real_buffer(buf) if real else buf))
    t1, t2 = _random_t(s, np.random.default_rng(34), real)
    p1, p2 = LR.pack_t1(s, t1), LR.pack_t2(s, t2)
    if real:
        p1, p2 = p1.real, p2.real
    d1, d2 = _dev(p1), _dev(p2)
    first = None
    for _ in range(20):
        r1, r2 = torch.full_like(d1, 3.0), torch.full_like(d2, 3.0)
        ctx.build_residual(d1, d2, r1, r2)
        got = r1.cpu(), r2.cpu()
        first = first or got
        assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1])
    R1, R2 = ccsd.residual(ccsd.Dense(s), t1, t2)
    scale = max(np.abs(R1).max(), np.abs(R2).max())
    for a, b in zip(first, (LR.pack_t1(s, R1), LR.pack_t2(s, R2))):
        assert np.abs(a.numpy() - b).max() <= 1e-12 * scale
    ctx.destroy()


@pytest.mark.parametrize("nocc,nvirt,nirrep", [(4, 16, 1), (6, 33, 2), (12, 26, 5)])
def test_imaginary_parts_of_nearly_real_residuals_keep_their_digits(nocc, nvirt, nirrep):
    """Imaginary parts 1e-9 of the real ones: each part of a product is summed by itself, so the imaginary parts of the
    residual are as good to their own size as the real ones (the bound of the tests above, per part)."""
    import torch
    import paper_2004_03682_amd as F
    small = 1e-9

    def shrink(x):
        return x.real + 1j * small * x.imag
    s = fsgen.make_system(nocc, nvirt, nirrep, 0.05, 93)
    ctx = F.Context.from_system(s)
    for C in fsgen.CLASSES:
        ctx.set_integrals(C, _dev(shrink(fsgen.class_buffer(s, C)[0])))
    t1, t2 = (shrink(t) for t in _random_t(s, np.random.default_rng(nvirt), False))
    d1, d2 = _dev(LR.pack_t1(s, t1)), _dev(LR.pack_t2(s, t2))
    r1, r2 = torch.empty_like(d1), torch.empty_like(d2)
    ctx.build_residual(d1, d2, r1, r2)
    be = ccsd.Dense(s)
    be.cls = {k: shrink(v) for k, v in be.cls.items()}
    R1, R2 = ccsd.residual(be, t1, t2)
    for part in (np.real, np.imag):
        scale = max(np.abs(part(R1)).max(), np.abs(part(R2)).max())
        for a, b in ((r1, LR.pack_t1(s, R1)), (r2, LR.pack_t2(s, R2))):
            assert np.abs(part(a.cpu().numpy()) - part(b)).max() <= 1e-12 * scale, part.__name__
    ctx.destroy()
