"""hp_residual against the oracle in both finest-level orders, with the result also where x or b stands.

Tolerance: each entry is one seven-point sum, 1e-13 relative as in test_gpu_parity; the returned
relative norm 1e-12.
"""
import numpy as np
import pytest

import oracle
from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [(80, 24, 40), (128, 16, 16), (36, 12, 7)])
@pytest.mark.parametrize("layout,place", [(1, "own"), (1, "x"), (1, "b"), (0, "own")])
def test_residual(n, layout, place):
    p = wl.polytrope(n, 0.01, seed=2)
    rng = np.random.default_rng(3)
    b, x = rng.standard_normal(p.shape), rng.standard_normal(p.shape)
    ref = oracle.residual(p.n, p.h, p.bc, p.rho, p.c2, p.dt, x, b).reshape(p.shape)
    with hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt) as s:
        if layout != s.get_option(hp.OPT_LAYOUT):
            if layout:
                pytest.skip("the grid has no split order")
            s.set_option(hp.OPT_LAYOUT, layout)
        bt, xt = dev(b), dev(x)
        r = {"own": torch.empty_like(bt), "x": xt, "b": bt}[place]
        rel = s.residual(bt, xt, r)
        torch.cuda.synchronize()
    assert np.linalg.norm(r.cpu().numpy() - ref) <= 1e-13 * np.linalg.norm(ref)
    assert abs(rel - np.linalg.norm(ref) / np.linalg.norm(b)) <= 1e-12 * rel
