"""What a solve and a V-cycle say when a barrier among the workgroups of a one-launch V-cycle or solve runs out of polls.

The wait is bounded, so such a launch ends and its z is worthless. Here the bound is set to 0 from the host: every
barrier counts as lost at once and every workgroup leaves in order (nothing hangs or faults). Solves have to end in
HP_EHIP in every mode that runs these launches, hp_precond has to give NaN, and the next calls have to be right
again. Whether helper workgroups join at all (else there is no barrier) depends on the GPU, so each
call is made until one does.
"""
import ctypes

import numpy as np
import pytest

from oracle import nn
from paper_1112_3507_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

import paper_1112_3507_amd as hp  # noqa: E402

DEV = "cuda:0"
WHOLE, PARTLY = (16, 16, 16), (64, 16, 32)
TRIES = 50


def polls(s, count):
    lib = hp.load_library()
    lib.hp_test_barrier_polls.argtypes = [ctypes.c_void_p, ctypes.c_int]
    lib.hp_test_barrier_polls.restype = None
    lib.hp_test_barrier_polls(s._h, count)


def problem(n):
    p = wl.polytrope(n, 0.05, seed=7)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    s = hp.setup(p.n, p.h, p.bc, dev(p.rho), dev(p.c2), p.dt)
    return s, dev(wl.rhs_white(n, 8))


def solve(s, b):
    x = torch.zeros_like(b)
    return s.solve(b, x, tol=1e-10, check=False), x


@pytest.mark.parametrize("n,mode,timing", [(WHOLE, hp.MODE_FP64_MGPCG, 0), (WHOLE, hp.MODE_FP64_MGPCG, 1),
                                           (PARTLY, hp.MODE_FP64_MGPCG, 0), (WHOLE, hp.MODE_LEARNED, 0),
                                           (PARTLY, hp.MODE_LEARNED, 0)])
def test_solves_end_in_an_error(n, mode, timing):
    s, b = problem(n)
    with s:
        net = hp.Net(n)
        net.set_params(torch.from_numpy(nn.init_params(3).astype(np.float32)).to(DEV))
        s.attach_net(net)
        s.set_option(hp.OPT_MODE, mode)
        s.set_option(hp.OPT_KERNEL_TIMING, timing)  # 1: solved launch by launch
        first, x0 = solve(s, b)
        assert first["converged"]
        polls(s, 0)
        codes = []
        while len(codes) < TRIES and hp.EHIP not in codes:
            codes.append(solve(s, b)[0]["rc"])
        assert codes[-1] == hp.EHIP and set(codes[:-1]) <= {hp.OK}, codes
        assert b"did not finish" in hp.load_library().hp_last_error()
        polls(s, 1 << 22)
        again, x1 = solve(s, b)
        assert again["rc"] == hp.OK and again["iterations"] == first["iterations"] and torch.equal(x0, x1)
        s.attach_net(None)
        net.close()


@pytest.mark.parametrize("n", [WHOLE, PARTLY])
def test_v_cycle_is_nan(n):
    s, b = problem(n)
    with s:
        z, lost = torch.empty_like(b), torch.empty_like(b)
        s.precond(b, z)
        polls(s, 0)
        for _ in range(TRIES):
            s.precond(b, lost)
            if not torch.equal(lost, z):
                break
        assert torch.isnan(lost).all()
        polls(s, 1 << 22)
        s.precond(b, lost)
        assert torch.equal(lost, z)
        assert solve(s, b)[0]["converged"]
