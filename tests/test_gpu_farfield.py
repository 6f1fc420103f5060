"""Far field and its adjoint as matrix products: row, direction and basis
counts around the edges of the kernels' 64 x 64 tiles and 8-wide steps,
directions that are not unit vectors, and calls that take several direction
groups, against the oracle's sums.

Tolerance 1e-12: a result sums at most n = 480 x 9 products, whose rounding
in any order is below n eps = 1e-12 of the sum of magnitudes in the worst
case and sqrt(n) eps = 1.5e-14 for random signs."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim, rel

pytestmark = pytest.mark.gpu
NAME, TOL = W.SPHERE_L2_NARROW.name, 1e-12


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.mark.parametrize("nd,nt,batch,scale", [(1, 1, 1, 1.0), (31, 13, 5, 1.0), (33, 64, 1, 1.0), (40, 3, 21, 1.0),
                                               (21, 9, 7, 1.25), (22, 7, 9, 0.5)])
def test_products_at_tile_edges(torch, nd, nt, batch, scale):
    from oracle import farfield
    print("far field: directions", nd, "steps", nt, "columns", batch, "scale", scale, flush=True)
    s, _, _, p = oracle_aim(NAME)
    dirs = W.unit_vectors(5, 4, nd)
    dirs[-1] *= scale
    F = farfield.FarField(s, dirs, p["dt"], W.SPHERE_L2_NARROW.f0)
    P = gpu_problem(NAME, nt=nt, batch=batch)
    I, Ub = W.complex_normal(3, (nt, batch, s.ns)), W.complex_normal(4, (nt, batch, nd, 3))
    U = P.farfield(dirs, torch.from_numpy(I).cuda()).cpu().numpy()
    S = P.farfield_adjoint(dirs, torch.from_numpy(Ub).cuda()).cpu().numpy()
    P.close()
    assert rel(U, F.apply(I)) < TOL
    assert rel(S, F.adjoint(Ub)) < TOL


def test_direction_groups(torch):
    # 2000 directions of this problem pass the tap table's bound
    print("far field: 2000 directions", flush=True)
    nt, batch = 3, 2
    dirs = W.unit_vectors(6, 4, 2000)
    P = gpu_problem(NAME, nt=nt, batch=batch)
    I = torch.from_numpy(W.complex_normal(7, (nt, batch, P.ns))).cuda()
    U = P.farfield(dirs, I)
    parts = torch.cat([P.farfield(dirs[a:a + 500], I) for a in range(0, 2000, 500)], 2)
    assert rel(U.cpu().numpy(), parts.cpu().numpy()) < TOL
    S = P.farfield_adjoint(dirs, U)
    parts = sum(P.farfield_adjoint(dirs[a:a + 500], U[:, :, a:a + 500].contiguous()) for a in range(0, 2000, 500))
    assert rel(S.cpu().numpy(), parts.cpu().numpy()) < TOL
    P.close()
