"""Coefficients far from 1: the coarsest inverse takes any positive finite operator, whatever its scale.

The density times 2^530 or 2^-530 (1e+-160) divides the operator by it, so coarsest solves and FP64 solves have to give
that multiple of what they give without it; and densities that are 2^-900 in every other cell, or at random, put
entries of such different sizes next to each other in one pivot block. Tolerance as for the coarsest
inverse elsewhere: 1e-10 relative; with mixed scales for the light cells and the heavy ones apart (scaled to a
unit diagonal that system is well conditioned, and the two hardly couple).
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


def coarse(p, b):
    x = torch.empty(p.shape, dtype=torch.float64, device="cuda:0")
    with hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt) as s:
        s.coarse_solve(dev(b), x)
    return x.cpu().numpy()


@pytest.mark.parametrize("power", [530, -530])
def test_scaled_operator(power):
    s = 2.0 ** power
    p = wl.polytrope((8, 8, 8), 0.02, seed=3)
    b = np.random.default_rng(4).standard_normal(p.shape)
    ref = coarse(p, b)
    x = coarse(dataclasses.replace(p, rho=p.rho * s), b) / s
    assert np.linalg.norm(x - ref) <= 1e-10 * np.linalg.norm(ref)
    p = wl.polytrope((16, 16, 16), 0.05, seed=7)
    b = wl.rhs_white(p.n, 8)
    out = []
    for f in (1.0, s):
        x = torch.zeros(p.shape, dtype=torch.float64, device="cuda:0")
        with hp.setup(p.n, p.h, p.bc, dev(p.rho * f), dev(p.c2), p.dt) as h:
            assert h.solve(dev(b), x, tol=1e-12)["converged"]
        out.append(x.cpu().numpy() / f)
    assert np.linalg.norm(out[1] - out[0]) <= 1e-10 * np.linalg.norm(out[0])


@pytest.mark.parametrize("kind", ["every other", "random"])
def test_mixed_scales(kind):
    n = (8, 8, 8)
    p = dataclasses.replace(wl.polytrope(n, 1.0, seed=3), bc=(P, P, N))
    light = (np.indices(p.shape).sum(0) % 2 == 1) if kind == "every other" else np.random.default_rng(5).random(p.shape) < 0.5
    p = dataclasses.replace(p, rho=np.where(light, 2.0 ** -900, 1.0), c2=np.ones(p.shape))
    A = mg.dense_operator(mg.build_hierarchy(p.n, p.h, p.bc, p.rho, p.c2, p.dt)[-1])
    b = np.random.default_rng(4).standard_normal(p.shape)
    # the reference by the system with a diagonal in [1, 4) (powers of two: nothing is rounded)
    scale = 2.0 ** -np.floor(np.log2(np.diag(A)) / 2)
    ref = (scale * np.linalg.solve(scale[:, None] * A * scale, scale * b.ravel())).reshape(p.shape)
    x = coarse(p, b)
    for part in (light, ~light):
        # (scaled before its norm: the square of 2^-900 is zero)
        f = 1.0 / np.abs(ref[part]).max()
        assert np.linalg.norm((x[part] - ref[part]) * f) <= 1e-10 * np.linalg.norm(ref[part] * f)
