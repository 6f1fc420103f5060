"""Far-field directions that are not finite, and directions a few rounding
errors off the unit sphere.

A direction with a NaN or an infinity gives a field that is not a number in
every component of that direction, and an adjoint that is not a number
anywhere (each of its sums takes the direction in); the other directions keep
their field.  A direction d with |d|^2 = 1 + e keeps the part -e d (d . f) that
I - d d leaves along d: e = 8e-13 here, against a rounding of the sums of
sqrt(480 x 9) eps = 1.5e-14, so 1e-13 tells the two apart."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import blif_of, gpu_problem, oracle_aim, rel

pytestmark = pytest.mark.gpu
WL = W.SPHERE_L2_NARROW
NAN, INF = float("nan"), float("inf")


@pytest.mark.parametrize("basis", [0, 1], ids=["cppif", "blif"])
@pytest.mark.parametrize("bad", [(NAN, 0.0, 0.0), (NAN, NAN, NAN), (0.0, 0.0, INF), (-INF, 0.6, 0.8), (INF, INF, INF)],
                         ids=str)
def test_direction_not_finite(bad, basis):
    import torch
    from oracle import farfield
    print("far field: direction", bad, "basis", basis, flush=True)
    s, _, _, p = oracle_aim(WL.name)
    nt, batch, at = 4, 2, 1
    dirs = W.unit_vectors(5, 4, 3)
    F = farfield.FarField(s, dirs, p["dt"], WL.f0, blif_of(WL, p["dt"])[0] if basis else None)
    dirs = np.insert(dirs, at, bad, axis=0)
    keep = [d for d in range(len(dirs)) if d != at]
    P = gpu_problem(WL.name, nt=nt, batch=batch, basis=basis)
    I = W.complex_normal(3, (nt, batch, s.ns))
    U = P.farfield(dirs, torch.from_numpy(I).cuda())
    S = P.farfield_adjoint(dirs, torch.from_numpy(W.complex_normal(4, (nt, batch, len(dirs), 3))).cuda())
    P.close()
    assert torch.isnan(torch.view_as_real(U[:, :, at])).all()
    assert rel(U[:, :, keep].cpu().numpy(), F.apply(I)) < 1e-12
    assert torch.isnan(torch.view_as_real(S)).all()


def test_direction_nearly_unit():
    import torch
    from oracle import farfield
    print("far field: directions nearly on the unit sphere", flush=True)
    s, _, _, p = oracle_aim(WL.name)
    nt, batch = 4, 2
    dirs = W.unit_vectors(5, 4, 3) * (1.0 + 4e-13)
    F = farfield.FarField(s, dirs, p["dt"], WL.f0)
    P = gpu_problem(WL.name, nt=nt, batch=batch)
    I, Ub = W.complex_normal(3, (nt, batch, s.ns)), W.complex_normal(4, (nt, batch, len(dirs), 3))
    U = P.farfield(dirs, torch.from_numpy(I).cuda()).cpu().numpy()
    S = P.farfield_adjoint(dirs, torch.from_numpy(Ub).cuda()).cpu().numpy()
    P.close()
    print("   rel", rel(U, F.apply(I)), rel(S, F.adjoint(Ub)), flush=True)
    assert rel(U, F.apply(I)) < 1e-13
    assert rel(S, F.adjoint(Ub)) < 1e-13
