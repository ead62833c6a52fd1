"""The forms a rate table is evaluated in, against the oracle on the same table:
fine steps with a small change per interval (the compiled-in fast forms), fine
steps with a large one (a grey table: tau P'/P reaches -80), and steps too
coarse for the series of the position.  Few sources (teams and single waves),
many small ones (groups) and many with kept records (pyramids from the lists),
and both adjoints.  Rates are FP32: an optical depth rounded to 6e-8 moves a
grey P by 80 times that, which sets the 1e-5."""
import math

import numpy as np
import pytest
import torch

import oracle
from tests.parity import assert_grad_parity, assert_parity
from workloads import make_workload

pytestmark = pytest.mark.gpu
TOL = 1e-5
TABLES = {
    "fine": lambda: oracle.blackbody_table(n=2600),
    "steep": lambda: oracle.grey_table(),
    "coarse": lambda: oracle.blackbody_table(n=300),
    "coarse-steep": lambda: oracle.grey_table(n=240, lg_lo=-8.0, lg_hi=math.log10(20.0)),
}


@pytest.mark.parametrize("table", list(TABLES))
@pytest.mark.parametrize("n_src,N,R_hi", [(5, 23, 9.7), (90, 18, 6.0), (1400, 16, 5.2), (700, 17, 7.9)])
def test_rates_and_gradients_against_oracle(table, n_src, N, R_hi):
    import paper_2311_01492_amd as asora
    print("case table", table, n_src, N, R_hi, flush=True)
    tb = TABLES[table]()
    w = make_workload("c2", N=N, n_src=n_src, R=(0.5, 1.0), seed=3 + n_src)
    rng = np.random.default_rng(n_src)
    w.src.ijk[:] = rng.integers(0, N, size=(n_src, 3)).astype(np.int32)
    w.src.R[:] = rng.uniform(0.0, R_hi, size=n_src).astype(np.float32)
    args = (w.N, w.cell_cm, tb, w.n_H, w.x_HI, w.src.ijk, w.src.Q, w.src.R)
    og = oracle.raytrace(*args)
    gbar = rng.standard_normal((N, N, N)) / (og.max() + 1e-300)
    on, ox, oq = oracle.raytrace_grad(*args, gbar)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    src = [t(a) for a in (w.n_H, w.x_HI, w.src.ijk, w.src.Q, w.src.R)]
    ctx = asora.Asora(w.N, w.cell_cm, tb.P, tb.dP, tb.lg_lo, tb.lg_hi, tau_w=0.6)
    assert_parity(ctx.raytrace(*src).cpu(), og, TOL)
    assert_parity(ctx.raytrace(*src, early_exit=True).cpu(), og, TOL, what="early exit")
    rec = ctx.backward(*src, t(gbar))
    assert_parity(ctx.raytrace(*src, store=True).cpu(), og, TOL, what="keeping forward")
    kept = ctx.backward(*src, t(gbar), store=True)
    ctx.check()
    for form, got in (("recomputed", rec), ("kept", kept)):
        for a, o, name in zip(got, (on, ox, oq), ("dn", "dx", "dQ")):
            assert_grad_parity(a.cpu(), o, TOL, what=f"{name}, {form}")
