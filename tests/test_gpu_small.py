"""V-cycles of small levels and whole FP64 solves of small grids, which run in one launch, against the oracle.

Grids at the edges of that rule: one to four cells of a colour per thread (512 threads), 2D, 3D and
semi-coarsened, odd and closed axes, both storage orders, the most cells (4096), a coarsest level
solved by the owner alone (<= 64 cells), by helpers, and of 1953 cells (odd sizes stop the coarsening);
an odd grid just too large; and grids of which only the lower levels are small.

Tolerances as in test_gpu_parity: V-cycle 1e-9 relative (the dense inverse against the oracle's solve),
solves 1e-9 relative L2 at a true relative residual of 1e-10.
"""
import dataclasses
import functools

import numpy as np
import pytest

import oracle
from oracle import mg
from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

DEV = "cuda:0"
P, N = hp.PERIODIC, hp.NEUMANN
WHOLE = [((64, 1, 64), (P, P, N)), ((16, 16, 16), (P, P, N)), ((66, 1, 62), (N, P, N)), ((63, 1, 62), (N, P, N)), ((45, 1, 90), (N, P, N)),
         ((64, 8, 8), (P, P, N)), ((13, 12, 26), (N, N, N)), ((12, 10, 8), (P, N, P)), ((4, 4, 36), (P, P, N)),
         ((130, 1, 8), (N, P, N))]
PARTLY = [((32, 16, 24), (P, P, N)), ((128, 1, 96), (N, P, N)), ((64, 16, 32), (P, P, P))]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def relerr(a, b):
    return float(np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b)))


@functools.lru_cache(maxsize=None)
def problem(n, bc):
    return dataclasses.replace(wl.polytrope(n, 0.05, seed=7), bc=bc)


@functools.lru_cache(maxsize=None)
def reference(n, bc, rule=0):
    p = problem(n, bc)
    b = wl.rhs_white(n, 8)
    x, st = oracle.reference_solve(p.n, p.h, p.bc, p.rho, p.c2, p.dt, b, face_rule=rule)
    assert st["converged"] or st["stagnated"]
    return b, x


def make(p):
    return hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt)


def check_solve(s, b, xref, start=None):
    x = torch.zeros(b.shape, dtype=torch.float64, device=DEV) if start is None else dev(start)
    st = s.solve(dev(b), x, tol=1e-10)
    assert st["converged"] and st["rel_residual"] <= 1e-10, st
    assert relerr(host(x), xref) <= 1e-9
    return st


@pytest.mark.parametrize("n,bc", WHOLE + PARTLY)
def test_vcycles_and_solves_match_oracle(n, bc):
    p = problem(n, bc)
    b, xref = reference(n, bc)
    rng = np.random.default_rng(9)
    r = rng.standard_normal(p.shape)
    with make(p) as s:
        default = s.get_option(hp.OPT_LAYOUT)
        for layout in dict.fromkeys((default, 0)):
            s.set_option(hp.OPT_LAYOUT, layout)
            for rule, pre, post in ((0, 1, 1), (1, 1, 2), (0, 2, 1)):
                s.set_option(hp.OPT_FACE_RULE, rule)
                s.set_option(hp.OPT_NU_PRE, pre)
                s.set_option(hp.OPT_NU_POST, post)
                lv = mg.build_hierarchy(p.n, p.h, p.bc, p.rho, p.c2, p.dt, coarsest_max=512, face_rule=rule)
                z = torch.empty(p.shape, dtype=torch.float64, device=DEV)
                s.precond(dev(r), z)
                assert relerr(host(z), mg.vcycle(lv, r, pre, post)) <= 1e-9, (layout, rule, pre, post)
            check_solve(s, b, xref)
            check_solve(s, b, xref, rng.standard_normal(p.shape))


def test_new_coefficients_and_repeats():
    (n, bc), rule = WHOLE[0], 1
    p = problem(n, bc)
    b, xref = reference(n, bc, rule)
    with make(dataclasses.replace(p, rho=p.rho[::-1] * 1.5)) as s:
        s.set_option(hp.OPT_FACE_RULE, rule)
        s.update_coefficients(dev(p.rho), dev(p.c2), p.dt)
        runs = []
        for _ in range(4):
            x = torch.zeros(p.shape, dtype=torch.float64, device=DEV)
            runs.append((s.solve(dev(b), x, tol=1e-10)["iterations"], host(x)))
        assert relerr(runs[0][1], xref) <= 1e-9
        # no value depends on how many helpers took part
        assert all(k == runs[0][0] and np.array_equal(x, runs[0][1]) for k, x in runs)


def test_ends_other_than_convergence():
    n, bc = WHOLE[1]
    p = problem(n, bc)
    b, xref = reference(n, bc)
    with make(p) as s:
        x = dev(np.ones(p.shape))
        st = s.solve(dev(np.zeros(p.shape)), x, tol=1e-10)
        assert st["converged"] and st["iterations"] == 0 and not host(x).any()
        bad = b.copy()
        bad[3, 2, 1] = np.inf
        for rhs, guess in ((bad, np.zeros(p.shape)), (b, np.where(bad == np.inf, np.nan, 0.0))):
            with pytest.raises(hp.HPError):
                s.solve(dev(rhs), dev(guess), tol=1e-10)
        # already solved: nothing to do
        x = dev(xref)
        assert s.solve(dev(b), x, tol=1e-10)["iterations"] == 0 and np.array_equal(host(x), xref)
        # the cap leaves the iterate and its residual
        s.set_option(hp.OPT_MAX_ITER, 3)
        x = torch.zeros(p.shape, dtype=torch.float64, device=DEV)
        st = s.solve(dev(b), x, tol=1e-10, check=False)
        assert st["rc"] == hp.ENOCONV and st["iterations"] == 3 and not st["converged"]
        r = oracle.residual(p.n, p.h, p.bc, p.rho, p.c2, p.dt, host(x), b)
        rel = np.linalg.norm(r) / np.linalg.norm(b)
        assert rel < 1.0 and abs(rel - st["rel_residual"]) <= 1e-6 * rel
        s.set_option(hp.OPT_MAX_ITER, 1000)
        check_solve(s, b, xref, host(x))
