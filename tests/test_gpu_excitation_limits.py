"""Excitation at the ends of the pulse width's and the delay's range, where a
quotient of the Gaussian has an infinite or subnormal divisor or overflows: an
infinite or huge width (a continuous wave), a width whose square is
subnormal and a pulse that is 1e160 s away (both zero at every step), against
the oracle.  Tolerance 1e-13 of the largest value, as in the other excitation
tests."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim

pytestmark = pytest.mark.gpu
WL = W.SPHERE_L2


@pytest.mark.parametrize("sigma,td,zero", [(float("inf"), WL.td, False), (1e160, WL.td, False),
                                           (1.2e154, WL.td, False), (1e-157, WL.td, True), (1e-150, WL.td, True),
                                           (WL.sigma, 1e160, True)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_limits(sigma, td, zero, noalloc):
    import torch
    from oracle import excitation
    print("excitation: sigma", sigma, "delay", td, "noalloc", noalloc, flush=True)
    nt, batch = 5, 2
    s, _, _, p = oracle_aim(WL.name)
    k = W.unit_vectors(2, 2, batch)
    pol = W.polarisations(2, k)
    P = gpu_problem(WL.name, nt=nt, batch=batch)
    V = torch.full((nt, batch, P.ns), 7.0, dtype=torch.complex128, device="cuda")
    P.excitation(k, pol, sigma, td, out=V, noalloc=noalloc)
    V = V.cpu().numpy()
    P.close()
    if zero:
        assert (V == 0).all()
        return
    with np.errstate(over="ignore"):
        ref = excitation.excitation(s, nt, p["dt"], k, pol, np.float64(sigma), td, WL.f0)
    assert np.isfinite(ref).all() and np.abs(V - ref).max() <= 1e-13 * np.abs(ref).max()
