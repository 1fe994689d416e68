"""Coefficients of every level where the finest level's setup and its coarsening are one pass, against the oracle.

The pass takes x pairs and one or two rows in y and z to a coarse cell, in natural and split order; odd x axes and
arrays that are not 16-byte aligned take two passes. Operators and diagonals (by one half sweep) of every level
1e-13 and 1e-12 relative as in test_gpu_parity; a bad cell anywhere is refused.
"""
import numpy as np
import pytest

from oracle import mg
from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402


def dev(a, off=0):
    t = torch.empty(a.size + off, dtype=torch.float64, device="cuda:0")[off:]
    t.copy_(torch.from_numpy(np.ascontiguousarray(a)).reshape(-1))
    return t.reshape(a.shape)


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("n", [(80, 24, 40), (128, 16, 16), (64, 1, 32), (48, 20, 1), (32, 8, 9), (30, 10, 20), (64, 10, 12)])
@pytest.mark.parametrize("two,off", [(False, 0), (True, 0), (False, 1)])
def test_levels(n, two, off):
    p = wl.polytrope(n, 0.01, seed=5)
    face = np.random.default_rng(6).uniform(0.5, 2.0, p.shape) if two else p.rho
    lv = mg.build_hierarchy(p.n, p.h, p.bc, p.rho, p.c2, p.dt, rho_face=face)
    rng = np.random.default_rng(7)
    with hp.setup(p.n, p.h, p.bc, dev(p.rho, off), dev(p.c2, off), p.dt,
                  rho_face=dev(face, off) if two else None) as s:
        assert s.num_levels() == len(lv)
        for l, L in enumerate(lv):
            x, r = rng.standard_normal(L.shape), rng.standard_normal(L.shape)
            y, z = torch.empty(L.shape, dtype=torch.float64, device="cuda:0"), dev(x)
            s.apply(l, dev(x), y)
            s.smooth(l, dev(r), z, 0)
            torch.cuda.synchronize()
            assert relerr(y.cpu().numpy(), mg.apply(L, x)) <= 1e-13, l
            assert relerr(z.cpu().numpy(), mg.half_sweep(L, r, x, 0)) <= 1e-12, l
        for cell, value in (((0, 0, 0), 0.0), (tuple(v - 1 for v in p.shape), np.nan)):
            bad = p.rho.copy()
            bad[cell] = value
            with pytest.raises(hp.HPError):
                s.update_coefficients(dev(bad, off), dev(p.c2, off), p.dt)
