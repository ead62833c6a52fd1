"""Calls of few sources take every source as pyramids in one launch, several
waves to a pyramid where the chip has room; calls of many take the sources from
sorted lists, small ones in groups of pyramids.  All of these, at the counts
where the number of waves to a pyramid changes (256 CUs: 7, 85, 170 sources),
where the lists begin (256, 512, 682 and 1365), where the groups change (to 24 pyramids at
3151) and where they come in beside pyramids or for shells (4096, 8192), on odd
and even grids and up to radii beyond half the box, against the shell sweeps of
the same sources.  Rates are FP32 in every form (1e-5, as against the oracle);
kept records and recomputed ones give the same FP64 sums, rounded once to the
FP32 outputs (1e-6)."""
import math

import numpy as np
import pytest
import torch

import oracle
from tests.parity import assert_grad_parity, assert_parity
from workloads import make_workload

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def asora():
    import paper_2311_01492_amd as m
    return m


def _inputs(N, n_src, R_hi, seed):
    w = make_workload("c2", N=N, n_src=n_src, R=(0.5, 1.0), seed=seed)
    rng = np.random.default_rng(seed)
    w.src.ijk[:] = rng.integers(0, N, size=(n_src, 3)).astype(np.int32)
    w.src.R[:] = rng.uniform(0.0, R_hi, size=n_src).astype(np.float32)
    w.src.R[0] = R_hi
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    gbar = t(rng.standard_normal((N, N, N)) * 1e12)
    return w, [t(a) for a in (w.n_H, w.x_HI, w.src.ijk, w.src.Q, w.src.R)], gbar


def _ctx(asora, w, heat=False, **kw):
    bb = oracle.blackbody_table()
    c = asora.Asora(w.N, w.cell_cm, bb.P, bb.dP, bb.lg_lo, bb.lg_hi, **kw)
    if heat:
        c.set_heating_table(*asora.table_blackbody_heat(lg_lo=bb.lg_lo, lg_hi=bb.lg_hi, n=len(bb.P))[:2])
    return c


def _np(x):
    return [a.cpu().numpy().astype(np.float64) for a in x]


@pytest.mark.parametrize("n_src,N,R_hi", [
    (1, 16, 0.9), (1, 17, 1.0), (1, 24, 18.0), (2, 23, 9.5), (7, 24, 11.9), (8, 21, 14.0), (85, 24, 5.0),
    (86, 25, 13.0), (170, 24, 11.0), (171, 25, 3.0), (256, 34, 16.1), (257, 34, 16.1), (512, 47, 22.9), (682, 20, 9.0), (683, 21, 9.0),
    (800, 20, 5.5), (800, 21, 9.7), (800, 33, 16.0),
    (1365, 16, 6.0), (4100, 20, 6.9), (1400, 18, 7.1), (1400, 29, 13.9), (3500, 26, 12.5), (4200, 48, 23.0), (8200, 50, 23.9)])
def test_every_count_against_shell_sweeps(asora, n_src, N, R_hi):
    print("case few sources", n_src, N, R_hi, flush=True)
    w, src, gbar = _inputs(N, n_src, R_hi, 31 + n_src)
    opt = dict(tau_w=0.6 if n_src % 2 else math.inf, halfpath_scalar=n_src % 3 == 0)
    a, b = _ctx(asora, w, heat=True, **opt), _ctx(asora, w, heat=True, **opt)
    b.set_tuning(pyramid_sweep=2)
    g, h = _np(a.raytrace_heating(*src))
    gs, hs = _np(b.raytrace_heating(*src))
    assert_parity(g, gs, TOL)
    assert_parity(h, hs, TOL, what="heating")
    assert_parity(_np([a.raytrace(*src, store=True)])[0], gs, TOL, what="keeping forward")
    kept = _np(a.backward(*src, gbar, store=True))
    assert_parity(_np([a.raytrace(*src, early_exit=True)])[0], gs, TOL, what="early exit")
    rec = _np(a.backward(*src, gbar))
    shell = _np(b.backward(*src, gbar))
    for x, y, z, name in zip(kept, rec, shell, ("dn", "dx", "dQ")):
        assert_grad_parity(x, y, 1e-6, what=name + ", kept against recomputed")
        assert_grad_parity(y, z, TOL, what=name)
    assert_parity(_np([a.raytrace_static(*src, out=torch.empty_like(src[0]))])[0], gs, TOL, what="static")
    if n_src == 1:
        (g1, c1), (g2, c2) = (_np(c.raytrace(*src, coldens=True)) for c in (a, b))
        assert_parity(g1, g2, TOL)
        np.testing.assert_allclose(c1, c2, rtol=1e-9, atol=1e-12 * c2.max())
    a.check()
    b.check()


def test_a_source_out_of_range_is_reported_and_skipped(asora):
    print("case few sources, one out of range", flush=True)
    w, src, gbar = _inputs(24, 5, 8.0, 5)
    c = _ctx(asora, w)
    good = src[:2] + [x[:4].contiguous() for x in src[2:]]
    want = [c.raytrace(*good, R_max=8.0)] + list(c.backward(*good, gbar, R_max=8.0))
    src[2][4, 1] = 24
    got = [c.raytrace(*src, R_max=8.0)] + list(c.backward(*src, gbar, R_max=8.0))
    with pytest.raises(asora.AsoraError):
        c.check()
    assert_parity(got[0].cpu(), want[0].cpu(), TOL)
    assert float(got[3][4]) == 0.0
    for x, y in zip(got[1:3] + [got[3][:4]], want[1:]):
        assert_grad_parity(x.cpu(), y.cpu(), 1e-6)
