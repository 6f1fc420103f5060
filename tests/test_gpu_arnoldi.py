"""GMRES on both sides of its launch rules: columns of one to eight entries
per thread of the one-launch orthogonalisation, basis sizes that pass its
bound within a cycle (the diagonal preconditioner takes many steps), restarts,
and columns that converge at different steps.  The first time step solves
Z_0 I = V; with the confirmed stop the true residual, formed here with the
library's product, meets the tolerance up to the rounding of the products
(1e-14 of ||V|| against a tolerance of 1e-8)."""
import dataclasses

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-8


@pytest.mark.parametrize("name,batch,restart", [("l2", 1, 60), ("l2", 3, 7), ("l3", 2, 60), ("plate", 1, 60),
                                                ("l4", 2, 20)])
def test_true_residual(name, batch, restart):
    import torch
    from paper_1408_7060_amd import FP64, Problem
    wl = {"l2": W.SPHERE_L2, "l3": W.SPHERE_L3, "l4": W.SPHERE_L4,
          "plate": dataclasses.replace(W.PLATE_1M, plate_size=3.0, grid=(24, 24, 8))}[name]
    print("gmres:", name, "columns", batch, "restart", restart, flush=True)
    xyz, tri, rwg = wl.mesh()
    kw = dict(ng=wl.ng) if wl.ng else dict(beta=wl.beta, f_bw=wl.f_bw)
    P = Problem(xyz, tri, rwg, fc=wl.f0, nt=1, grid=wl.grid, d_near=wl.near_lambda * W.C0 / wl.f0, precision=FP64,
                batch=batch, tol=TOL, restart=restart, maxit=4000, sync_every=3, **kw)
    P.set_tuning(dict(P.tuning(), precond=0))
    V = torch.from_numpy(W.complex_normal(9, (1, batch, P.ns))).cuda()
    V[:, -1] *= 1e-6   # a column of another scale
    V[:, 0, P.ns // 2:] = 0.0
    I, st = P.march(V)
    r = V[0] - P.apply_z(0, I[0])
    P.close()
    assert st["first_noconv_step"] < 0 and st["max_iters"] > 8
    assert float((r.norm(dim=1) / V[0].norm(dim=1)).max()) <= TOL * (1 + 1e-5)
