"""The coarsest operator's inverse at the edges of its order of elimination, against the oracle's solve.

One-level grids (at most 512 cells): layers along each axis, rings of layers (periodic) with an even and an odd
number of them, thin layers taken together, layers cut into several and into unequal blocks, a single
layer, padded blocks, and the smallest grids. Tolerance as in test_gpu_parity: 1e-10 relative.
"""
import dataclasses

import numpy as np
import pytest

from oracle import mg
from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

P, N = hp.PERIODIC, hp.NEUMANN


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n,bc", [
    ((8, 8, 8), (P, P, N)), ((16, 16, 2), (P, P, N)), ((6, 30, 2), (P, P, N)), ((16, 1, 32), (P, P, N)),
    ((100, 2, 2), (P, P, N)), ((2, 2, 100), (P, P, N)), ((5, 7, 11), (N, N, N)), ((22, 1, 23), (N, P, N)),
    ((2, 16, 16), (P, P, P)), ((34, 2, 7), (P, N, N)), ((512, 1, 1), (P, P, N)), ((1, 1, 7), (P, P, N)),
    ((1, 1, 1), (N, N, N)), ((2, 2, 2), (P, P, P)), ((17, 1, 2), (N, P, N))])
@pytest.mark.parametrize("rule", [0, 1])
def test_inverse_in_every_order(n, bc, rule):
    p = dataclasses.replace(wl.polytrope(n, 0.02, seed=3), bc=bc)
    L = mg.build_hierarchy(p.n, p.h, p.bc, p.rho, p.c2, p.dt, face_rule=rule)[-1]
    assert L.n == n
    b = np.random.default_rng(4).standard_normal(p.shape)
    x = torch.empty(p.shape, dtype=torch.float64, device="cuda:0")
    with hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt) as s:
        s.set_option(hp.OPT_FACE_RULE, rule)
        s.update_coefficients(dev(p.rho), dev(p.c2), p.dt)  # the workspace is used again
        s.coarse_solve(dev(b), x)
    torch.cuda.synchronize()
    ref = mg.coarse_solve(L, b)
    assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-10 * np.linalg.norm(ref)
