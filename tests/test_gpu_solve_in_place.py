"""Solves whose p shares memory with rhs, on grids in split storage order (there the library works on copies of both).

One grid that is solved in one launch (64 x 8 x 8 = 4096 cells, where the launch updates p itself) and one just above;
rhs and p the same array, and overlapping in part from either side. The same input from arrays apart has to
give the same bits: no value depends on where the arrays lie. And what both say of a solve that breaks down
(an initial guess whose residual's square overflows): the same code, iteration and residual, which is none.
"""
import numpy as np
import pytest

from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("n", [(64, 8, 8), (64, 16, 8)])
@pytest.mark.parametrize("rhs_at,p_at", [(0, 0), (0, 1111), (1111, 0)])
def test_p_on_rhs(n, rhs_at, p_at):
    p = wl.polytrope(n, 0.05, seed=7)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    cells = p.ncells
    memory = dev(np.random.default_rng(3).standard_normal(2 * cells))
    rhs, x = memory[rhs_at:rhs_at + cells], memory[p_at:p_at + cells]
    rhs_apart, x_apart = rhs.clone(), x.clone()
    with hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt) as s:
        assert s.get_option(hp.OPT_LAYOUT) == 1
        apart = s.solve(rhs_apart, x_apart, tol=1e-10)
        shared = s.solve(rhs, x, tol=1e-10, check=False)
    assert shared["rc"] == hp.OK and shared["converged"], shared
    assert shared["iterations"] == apart["iterations"]
    assert torch.equal(x, x_apart)


@pytest.mark.parametrize("n", [(64, 8, 8), (64, 16, 8)])
def test_breakdown_leaves_no_residual(n):
    p = wl.polytrope(n, 0.05, seed=7)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    x = dev(1e200 * np.random.default_rng(3).standard_normal(p.shape))
    with hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt) as s:
        st = s.solve(dev(wl.rhs_white(n, 8)), x, tol=1e-10, check=False)
    assert st["rc"] == hp.EBREAKDOWN and st["iterations"] == 1 and not st["converged"]
    assert st["rel_residual"] == 0.0
