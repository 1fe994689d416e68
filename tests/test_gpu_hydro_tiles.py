"""The explicit step and the passes around the solve at the edges of their column tiles and chunks.

Reference: the NumPy formulas of the oracle in FP64. A cell's result is its value plus dt times at
most six fluxes, each a handful of FP64 operations on values of the field's size, with dt |u| / h
under 1: 64 units in the last place of the largest value of the field bound the difference.
"""
import numpy as np
import pytest

from oracle import hydro, stepper

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

P, N = hp.PERIODIC, hp.NEUMANN
EPS = float(np.finfo(np.float64).eps)


def _close(got, ref, scale=None):
    ref = np.asarray(ref)
    got = got.cpu().numpy().reshape(ref.shape)
    size = np.max(np.abs(ref)) if scale is None else scale
    assert np.max(np.abs(got - ref)) <= 64 * EPS * size


# the smallest wraps; one-cell axes; tiles of 32 and of 64 columns with one cell over, closed and
# periodic; chunks of two planes with a remainder; rows past the last tile; a box of several tiles
@pytest.mark.parametrize("n,bc", [
    ((2, 2, 2), (P, P, P)), ((1, 12, 9), (P, P, N)), ((12, 1, 7), (N, P, N)), ((34, 18, 3), (P, P, N)),
    ((33, 9, 5), (N, N, N)), ((66, 10, 6), (P, P, P)), ((65, 17, 4), (N, N, N)), ((128, 34, 11), (P, P, N)),
])
def test_tiles_match_formulas(n, bc):
    rng = np.random.default_rng(sum(n))
    shape = n[::-1]
    h = (0.1, 0.13, 0.07)
    dt = 0.02
    rho = 1.0 + 0.5 * rng.random(shape)
    mom = rng.uniform(-1.0, 1.0, (3,) + shape)
    e = 2.0 + rng.random(shape)
    c2 = 1.0 + rng.random(shape)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    new = lambda *lead: torch.empty(lead + shape, dtype=torch.float64, device="cuda")  # noqa: E731
    with hp.setup(n, h, bc, d(rho), d(c2), dt) as s:
        r1, m1, e1 = new(), new(3), new()
        s.advect(d(rho), d(mom), d(e), r1, m1, e1)
        ref = stepper.advect(n, h, bc, dt, rho, mom, e)
        for got, want, field in zip((r1, m1, e1), ref, (rho, mom, e)):
            _close(got, want, max(np.max(np.abs(want)), np.max(np.abs(field))))
        p = 1.0 + rng.random(shape)
        rf = ref[0] + 1.0  # positive
        b = new()
        s.pressure_rhs(d(rho), d(c2), d(p), d(mom), d(rf), d(ref[1]), b)
        _close(b, hydro.pressure_rhs(n, h, bc, dt, rho, c2, p, mom, rf, ref[1]), 2.0)
        mo, uf, eo = new(3), new(3), new()
        s.pressure_update(d(p), d(rf), d(ref[1]), d(ref[2]), mo, uf, eo)
        for got, want in zip((mo, uf, eo), hydro.pressure_update(n, h, bc, dt, p, rf, ref[1], ref[2])):
            _close(got, want, max(np.max(np.abs(want)), 4.0))
