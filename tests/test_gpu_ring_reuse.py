"""Marches on rings that hold an earlier march: nothing of it is read, also
where the earlier history is not finite, and a state saved before the rings
are full holds zeros in the slots of the steps not marched.  Every y/z engine,
time blocks and multilevel time blocks; results bit-identical to a fresh
context's."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("grid,yz,mode", [(16, 2, 0), (16, 1, 0), (16, 0, 0), (16, 3, 0), (16, 2, 1), (18, 0, 0)])
def test_second_march(grid, yz, mode, precision):
    import torch
    print("ring reuse: grid", grid, "engine", yz, "mode", mode, "precision", precision, flush=True)
    nt = 9
    wl = W.SPHERE_L2

    def fresh():
        P = gpu_problem(wl.name, precision=precision, batch=2, nt=nt, grid=grid, tol=1e-6, flags=1)
        P.set_tuning(dict(P.tuning(), yz_engine=yz))
        P.set_delay_mode(mode)
        return P
    V = torch.from_numpy(W.complex_normal(5, (nt, 2, 480))).cuda()
    P, F = fresh(), fresh()
    hist = torch.full((P.info["ng"], 2, P.ns), float("nan"), dtype=torch.complex128, device="cuda")
    P.delayed_field(hist)
    for n in (2, nt):
        a, b = P.march(V, nsteps=n)[0][:n], F.march(V, nsteps=n)[0][:n]
        assert torch.equal(a, b)
        assert np.array_equal(P.save_state()[64:], F.save_state()[64:])
    P.march(V, nsteps=2)
    F.close()
    F = fresh()
    F.march(V, nsteps=2)
    assert np.array_equal(P.save_state()[64:], F.save_state()[64:])
    P.close()
    F.close()
