"""The far field's tap table where its taps are shared between threads (every
tap on its own, two or three threads for all of them) and where they are not,
for both temporal bases, against the oracle (1e-12, as in the other far-field
tests); and the BLIF's time, whose table once took ten times the CPPIF's call:
at most three times it, the smallest of ten calls each."""
import time

import pytest

import workloads as W
from gpu_cases import blif_of, gpu_problem, oracle_aim, rel

pytestmark = pytest.mark.gpu
WL = W.SPHERE_L2


@pytest.mark.parametrize("basis", [0, 1], ids=["cppif", "blif"])
@pytest.mark.parametrize("nd,scale", [(1, 1.0), (20, 1.0), (60, 1.0), (150, 1.0), (20, 0.75)])
def test_shared_taps(nd, scale, basis):
    import torch
    from oracle import farfield
    print("tap table: directions", nd, "scale", scale, "basis", basis, flush=True)
    s, _, _, p = oracle_aim(WL.name)
    nt, batch = 6, 1
    dirs = W.unit_vectors(5, 4, nd)
    dirs[-1] *= scale
    F = farfield.FarField(s, dirs, p["dt"], WL.f0, blif_of(WL, p["dt"])[0] if basis else None)
    P = gpu_problem(WL.name, nt=nt, batch=batch, basis=basis)
    I, Ub = W.complex_normal(3, (nt, batch, s.ns)), W.complex_normal(4, (nt, batch, nd, 3))
    U = P.farfield(dirs, torch.from_numpy(I).cuda()).cpu().numpy()
    S = P.farfield_adjoint(dirs, torch.from_numpy(Ub).cuda()).cpu().numpy()
    P.close()
    assert rel(U, F.apply(I)) < 1e-12
    assert rel(S, F.adjoint(Ub)) < 1e-12


def test_blif_time():
    import torch
    best = []
    for basis in (0, 1):
        P = gpu_problem(WL.name, nt=20, batch=1, basis=basis)
        I = torch.from_numpy(W.complex_normal(3, (20, 1, P.ns))).cuda()
        dirs = W.unit_vectors(5, 4, 9)
        t = []
        for _ in range(12):
            torch.cuda.synchronize()
            a = time.perf_counter()
            P.farfield(dirs, I)
            t.append(time.perf_counter() - a)
        P.close()
        best.append(min(t[2:]))
    print("far field: CPPIF", best[0], "BLIF", best[1], flush=True)
    assert best[1] <= 3.0 * best[0]
