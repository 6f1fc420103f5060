"""Excitation at the edges of its launch: one and several steps per thread,
step groups that do not divide N_t, basis groups that do not divide 256,
against the oracle.  Tolerance 1e-13 of the largest step: the phases
w (r.k/c + t_d), about 120 rad here, carry 120 eps = 2.7e-14, and the 14 terms
of a value add to less than 14 times their rounding."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,batch", [(1, 1), (7, 2), (91, 7), (70, 33), (129, 70)])
def test_steps_per_thread(nt, batch):
    import torch
    from oracle import excitation
    wl = W.SPHERE_L2
    print("excitation: steps", nt, "columns", batch, flush=True)
    s, _, _, p = oracle_aim(wl.name)
    k = W.unit_vectors(2, 2, batch)
    pol = W.polarisations(2, k)
    P = gpu_problem(wl.name, nt=nt, batch=batch)
    V = torch.full((nt, batch, P.ns), float("nan"), dtype=torch.complex128, device="cuda")
    P.excitation(k, pol, wl.sigma, wl.td, out=V)
    V = V.cpu().numpy()
    P.close()
    for b in sorted({0, batch // 2, batch - 1}):
        ref = excitation.excitation(s, nt, p["dt"], k[b], pol[b], wl.sigma, wl.td, wl.f0)[:, 0]
        assert np.abs(V[:, b] - ref).max() <= 1e-13 * np.abs(ref).max()
