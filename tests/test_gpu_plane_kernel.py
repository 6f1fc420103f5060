"""Products on every grid with a plane kernel of its own (k_plane_green), with
its x lines: cubes 18 to 96 and flat grids, one and three columns, both
precisions, against the oracle's FFT product, and the transposed (conjugate)
spectra through the adjoint march's solve.  Tolerances as the other operator
tests: 1e-12 in FP64; 1e-5 in FP32."""
import functools

import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, rel
from oracle import physics as ph

pytestmark = pytest.mark.gpu
GRIDS = [18, 27, 32, 36, 54, 64, 96, (32, 16, 8), (18, 24, 8), (16, 48, 8), (16, 96, 8), (24, 32, 32), (16, 36, 18)]


def _workload(grid):
    # grid spacings of a third of an edge and more: where a basis spans many
    # nodes the exact moments need huge weights, and the product (of any
    # implementation) loses digits to their cancellation
    return W.SPHERE_L2 if np.max(grid) < 54 or np.min(grid) == 8 else W.sweep_workload(4, 2.0, grid, 30)


@functools.lru_cache(maxsize=1)
def _oracle(grid):
    from oracle import aim, geometry
    wl = _workload(grid)
    xyz, tri, rwg = wl.mesh()
    dt = ph.dt_from_beta(wl.beta, wl.f_bw)
    s = geometry.Surface(xyz, tri, rwg)
    return wl, s, aim.AIM(s, grid, wl.near_lambda * ph.C0 / wl.f0, dt, wl.f0, ph.ng_from(ph.rmax_of(xyz), dt))


@pytest.mark.parametrize("grid", GRIDS, ids=str)
def test_product(grid, monkeypatch):
    import torch
    from oracle import aim
    from paper_1408_7060_amd import Problem
    monkeypatch.setattr(aim, "FFT_WORKERS", 8)
    wl, s, A = _oracle(grid)
    x = W.complex_normal(3, (3, s.ns))
    # the far part by the oracle, the near zone's values (not under test) as exported
    far = {m: A.far_matvec(m, x[2], direct=False) for m in (0, A.ng)}
    xyz, tri, rwg = wl.mesh()
    for precision, tol in ((0, 1e-12), (1, 1e-5)):
        for batch in (1, 3):
            print("plane kernel: grid", grid, "precision", precision, "columns", batch, flush=True)
            P = Problem(xyz, tri, rwg, fc=wl.f0, nt=1, grid=grid, d_near=wl.near_lambda * ph.C0 / wl.f0, beta=wl.beta,
                        f_bw=wl.f_bw, precision=precision, batch=batch)
            near, ptr, col = P.export("near"), P.export("rowptr"), P.export("col")
            xb = x[2:] if batch == 1 else x
            for m, f in far.items():
                ref = f.copy()
                if m <= P.info["mn"]:
                    ref += np.add.reduceat(near[m] * x[2][col], ptr[:-1])
                y = P.apply_z(m, torch.from_numpy(xb).cuda()).cpu().numpy()[-1]
                assert rel(y, ref) <= tol
            P.close()


@pytest.mark.parametrize("grid", [18, 32, (18, 24, 8)], ids=str)
def test_adjoint_identity(grid):
    # <Z0^-H S, V> = <S, Z0^-1 V> with the solver's tolerance
    import torch
    print("plane kernel: adjoint, grid", grid, flush=True)
    P = gpu_problem(W.SPHERE_L2.name, batch=2, grid=grid, nt=1, tol=1e-12)
    V, S = (torch.from_numpy(W.complex_normal(k, (1, 2, P.ns))).cuda() for k in (4, 5))
    I, L = P.march(V)[0], P.adjoint_march(S)[0]
    P.close()
    for b in range(2):
        lhs, rhs = torch.vdot(L[0, b], V[0, b]), torch.vdot(S[0, b], I[0, b])
        assert abs(lhs - rhs) <= 1e-9 * float(S[0, b].norm() * I[0, b].norm())
