"""The passes around the solve on boxes of at most four rows, which lie in a tile whole, and on single planes.

Every number of such rows, closed and periodic (two rows: a cell's both neighbours are the same one, and the advection
reaches round to the cell itself), x of one cell, one tile of 64 columns, one cell short of it and over it, and of three
tiles; z of one plane, a chunk of two, and chunks with a remainder. Planes (more rows, nz = 1) with tiles of 32 x 8 cut
by the box. Then boxes at the edges of the rule for the length of chunks. Reference and bound as in test_gpu_hydro_tiles: 64 units in the last place of the largest term.
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
BOXES = [((64, 1, 7), (P, P, N)), ((65, 1, 1), (N, P, N)), ((1, 1, 9), (P, P, N)), ((130, 1, 2), (P, N, P)),
         ((66, 2, 5), (P, P, N)), ((63, 2, 2), (N, N, N)), ((2, 2, 6), (P, P, P)), ((129, 3, 5), (N, N, N)),
         ((64, 3, 1), (P, N, N)), ((1, 3, 4), (P, N, N)), ((66, 4, 6), (P, P, P)), ((65, 4, 3), (N, N, N)),
         ((3, 4, 5), (N, P, N)), ((34, 10, 1), (P, P, P)), ((33, 5, 1), (N, N, N)), ((64, 17, 1), (P, N, P)),
         ((64, 4, 300), (P, P, N))]
# where chunks get longer: 4096 planes of tiles (8 to a chunk), some more with a remainder, 16 to a chunk with one
CHUNKS = [((64, 64, 256), (P, P, N)), ((96, 80, 148), (P, P, N)), ((128, 64, 260), (P, N, N)), ((1024, 4, 522), (P, P, N))]


def _close(got, ref, scale):
    ref = np.asarray(ref)
    got = got.cpu().numpy().reshape(ref.shape)
    assert np.max(np.abs(got - ref)) <= 64 * EPS * scale


@pytest.mark.parametrize("n,bc", BOXES + CHUNKS)
def test_passes_match_formulas(n, bc):
    rng = np.random.default_rng(sum(n))
    shape = n[::-1]
    h, dt = (0.1, 0.13, 0.07), 0.02
    draw = lambda low, high, *lead: rng.uniform(low, high, lead + shape)  # noqa: E731
    rho, c2, p, e = draw(1, 1.5), draw(1, 2), draw(1, 2), draw(2, 3)
    mom, visc, temp, conc, rkc = draw(-1, 1, 3), draw(-1, 1), draw(1, 2), draw(0, 1), draw(0.01, 0.02)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    new = lambda *lead: torch.empty(lead + shape, dtype=torch.float64, device="cuda")  # noqa: E731
    with hp.setup(n, h, bc, d(rho), d(c2), dt) as s:
        out = new(), new(3), new()
        s.advect(d(rho), d(mom), d(e), *out)
        star = stepper.advect(n, h, bc, dt, rho, mom, e)
        for got, want, field in zip(out, star, (rho, mom, e)):
            _close(got, want, max(np.max(np.abs(want)), np.max(np.abs(field))))
        rf = star[0] + 1.0  # positive
        b = new()
        # the two-component term: at most six fluxes of rkc / h^2 (both terms of the rest are below 2)
        two = 0.75 * dt * np.max(temp) / np.min(rho * c2) * 2 * np.max(rkc) * sum(1 / q ** 2 for q in h)
        for opt in ({}, {"visc": visc}, {"temp_n": temp, "conc_n": conc, "rkc_n": rkc},
                    {"visc": visc, "temp_n": temp, "conc_n": conc, "rkc_n": rkc}):
            s.pressure_rhs(d(rho), d(c2), d(p), d(mom), d(rf), d(star[1]), b, **{k: d(v) for k, v in opt.items()})
            _close(b, hydro.pressure_rhs(n, h, bc, dt, rho, c2, p, mom, rf, star[1], r_gas=1.0, **opt), 2.0 + two)
        out = new(3), new(3), new()
        s.pressure_update(d(p), d(rf), d(star[1]), d(star[2]), *out)
        for got, want in zip(out, hydro.pressure_update(n, h, bc, dt, p, rf, star[1], star[2])):
            _close(got, want, max(np.max(np.abs(want)), 4.0))
