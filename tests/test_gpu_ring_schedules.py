"""Marches on rings that hold an earlier history (all of it NaN), in the
schedules that read them differently: history depths of one to four chunks of
the time-block pass with blocks that start inside the first chunk and past it,
one column (the single-plane delayed kernel), three levels and more of
multilevel time blocks, the CFIE's second pass, the adjoint march and
replayed whole steps.  Bit-identical to a fresh context's march."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import params_of

pytestmark = pytest.mark.gpu
F_CONTINUE, F_IMPLICIT_STOP, F_STEP_GRAPH = 1, 8, 32


def _problem(ng, nt, batch, precision, yz, mode, alpha=1.0, flags=F_CONTINUE, grid=16):
    from paper_1408_7060_amd import Problem
    wl = W.SPHERE_L2
    p = params_of(wl)
    P = Problem(p["xyz"], p["tri"], p["rwg"], fc=wl.f0, nt=nt, grid=grid, d_near=p["d_near"], ng=ng, f_bw=wl.f_bw,
                precision=precision, batch=batch, tol=1e-6, restart=60, maxit=300, flags=flags, sync_every=4,
                alpha=alpha)
    P.set_tuning(dict(P.tuning(), yz_engine=yz))
    P.set_delay_mode(mode)
    return P


def _stale(P, torch):
    P.delayed_field(torch.full((P.info["ng"], P.batch, P.ns), float("nan"), dtype=torch.complex128, device="cuda"))
    return P


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ng,batch,yz,mode,alpha", [
    (12, 1, 2, 0, 1.0), (20, 1, 2, 0, 1.0), (20, 2, 1, 0, 1.0), (30, 2, 2, 0, 1.0), (20, 1, 3, 0, 1.0),
    (30, 2, 3, 0, 1.0), (20, 1, 0, 0, 1.0), (40, 1, 2, 1, 1.0), (40, 2, 0, 1, 1.0), (26, 1, 3, 1, 1.0),
    (20, 2, 2, 0, 0.5), (20, 1, 3, 0, 0.5), (14, 1, 2, 1, 0.5)])
def test_forward(ng, batch, yz, mode, alpha, precision):
    import torch
    print("stale rings: N_g", ng, "columns", batch, "engine", yz, "mode", mode, "alpha", alpha, "precision", precision,
          flush=True)
    nt = 27
    V = torch.from_numpy(W.complex_normal(5, (nt, batch, 480))).cuda()
    P = _stale(_problem(ng, nt, batch, precision, yz, mode, alpha), torch)
    F = _problem(ng, nt, batch, precision, yz, mode, alpha)
    for n in (3, nt):
        a, b = P.march(V, nsteps=n)[0][:n], F.march(V, nsteps=n)[0][:n]
        assert torch.isfinite(torch.view_as_real(a)).all()
        assert torch.equal(a, b)
        assert np.array_equal(P.save_state()[64:], F.save_state()[64:])
        _stale(P, torch)
    P.close()
    F.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ng,batch,yz,mode", [(20, 1, 2, 0), (30, 2, 2, 0), (20, 1, 3, 0), (14, 2, 2, 1)])
def test_adjoint(ng, batch, yz, mode, precision):
    import torch
    print("stale rings, adjoint: N_g", ng, "columns", batch, "engine", yz, "mode", mode, "precision", precision,
          flush=True)
    nt = 27
    S = torch.from_numpy(W.complex_normal(6, (nt, batch, 480))).cuda()
    P, F = _stale(_problem(ng, nt, batch, precision, yz, mode), torch), _problem(ng, nt, batch, precision, yz, mode)
    a, b = P.adjoint_march(S)[0], F.adjoint_march(S)[0]
    assert torch.isfinite(torch.view_as_real(a)).all()
    assert torch.equal(a, b)
    P.close()
    F.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("ng,batch", [(12, 1), (20, 1), (20, 2), (30, 1)])
def test_step_graphs(ng, batch, precision):
    import torch
    print("stale rings, step graphs: N_g", ng, "columns", batch, "precision", precision, flush=True)
    nt, flags = 40, F_CONTINUE | F_IMPLICIT_STOP | F_STEP_GRAPH
    V = torch.from_numpy(W.complex_normal(5, (nt, batch, 480))).cuda()
    E = _problem(ng, nt, batch, precision, 2, 0, flags=F_CONTINUE | F_IMPLICIT_STOP)
    ref = E.march(V)[0]
    E.close()
    P = _problem(ng, nt, batch, precision, 2, 0, flags=flags)
    for _ in range(2):
        I, st = P.march(V)
        assert st["graph_steps"] > 0
        assert torch.isfinite(torch.view_as_real(I)).all()
        assert torch.equal(I, ref)
        _stale(P, torch)
    P.close()
