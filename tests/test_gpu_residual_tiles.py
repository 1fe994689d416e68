"""hp_residual, and the diagonals by one half sweep, where the 128 x 4 column tiles end within or beside the grid,
closed and periodic.

Tolerance: each entry is one seven-point sum of values of order 1, 1e-13 relative as in
test_gpu_parity; the returned relative norm and the half sweep 1e-12.
"""
import numpy as np
import pytest

import oracle
from oracle import mg

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402


@pytest.mark.parametrize("n", [(64, 4, 8), (126, 6, 12), (128, 8, 16), (130, 6, 10), (192, 12, 18), (256, 10, 34)])
@pytest.mark.parametrize("bc", [(hp.PERIODIC, hp.PERIODIC, hp.NEUMANN), (hp.NEUMANN, hp.PERIODIC, hp.NEUMANN),
                                (hp.PERIODIC, hp.NEUMANN, hp.PERIODIC), (hp.NEUMANN, hp.NEUMANN, hp.PERIODIC)])
def test_residual_tiles(n, bc):
    rng = np.random.default_rng(7)
    shape = n[::-1]
    rho, c2 = 1.0 + rng.random(shape), 1.0 + rng.random(shape)
    b, x = rng.standard_normal(shape), rng.standard_normal(shape)
    h, dt = (0.1, 0.2, 0.3), 0.5
    ref = np.asarray(oracle.residual(n, h, bc, rho, c2, dt, x, b)).reshape(shape)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    with hp.setup(n, h, bc, dev(rho), dev(c2), dt) as s:
        r = torch.empty(shape, dtype=torch.float64, device="cuda")
        rel = s.residual(dev(b), dev(x), r)
        torch.cuda.synchronize()
    assert np.linalg.norm(r.cpu().numpy() - ref) <= 1e-13 * np.linalg.norm(ref)
    assert abs(rel - np.linalg.norm(ref) / np.linalg.norm(b)) <= 1e-12 * rel


@pytest.mark.parametrize("n", [(64, 4, 8), (126, 6, 12), (128, 8, 16), (130, 6, 10), (65, 6, 9)])
@pytest.mark.parametrize("bc", [(hp.NEUMANN, hp.PERIODIC, hp.NEUMANN), (hp.PERIODIC, hp.NEUMANN, hp.NEUMANN),
                                (hp.NEUMANN, hp.NEUMANN, hp.NEUMANN)])
def test_diagonal_tiles(n, bc):
    if n[0] % 2 and bc[0] == hp.PERIODIC:
        pytest.skip("periodic axes have an even number of cells")
    rng = np.random.default_rng(8)
    shape = n[::-1]
    rho, c2 = 1.0 + rng.random(shape), 1.0 + rng.random(shape)
    h, dt = (0.1, 0.2, 0.3), 0.5
    L = mg.build_hierarchy(n, h, bc, rho, c2, dt)[0]
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    with hp.setup(n, h, bc, dev(rho), dev(c2), dt) as s:
        for colour in (0, 1):
            x, r = rng.standard_normal(shape), rng.standard_normal(shape)
            z = dev(x.copy())
            s.smooth(0, dev(r), z, colour)
            torch.cuda.synchronize()
            ref = mg.half_sweep(L, r, x, colour)
            assert np.linalg.norm(z.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref), colour
