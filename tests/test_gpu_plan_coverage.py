"""Radix plans and LDS passes where launches depend on them: the commit and
the delayed field of the 18^3 grid (whose products run on register lines and
the plane kernel), and products on grids with neither (12^3 and 9 x 12 x 8),
along each axis and on both the plane passes and the line passes, against the
oracle.  Tolerance 1e-12 as in the other FP64 operator tests."""
import functools

import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim, oracle_matvec, rel
from test_gpu_schedule import _plans

pytestmark = pytest.mark.gpu


def _try(P, d):
    try:
        P.set_tuning(d)
    except Exception as e:  # the plan does not fit the register staging
        assert getattr(e, "code", None) == -7, e
        return False
    return True


@pytest.mark.parametrize("yz", [0, 3])
def test_history_plans(yz):
    import torch
    name = W.SPHERE_L3.name
    s, A, _, p = oracle_aim(name)
    P = gpu_problem(name, nt=8)
    base = dict(P.tuning(), yz_engine=yz)
    hist = W.complex_normal(31, (p["ng"], 1, s.ns))
    ref = sum(oracle_matvec(name, m, hist[m - 1], direct=False) for m in range(1, p["ng"] + 1))
    h = torch.from_numpy(hist).cuda()
    tried = 0
    for pl in _plans(36, 3):
        if not _try(P, dict(base, radix_y=pl, radix_z=pl)):
            continue
        print("history plans: engine", yz, "plan", pl, flush=True)
        assert rel(P.delayed_field(h).cpu().numpy(), ref) <= 1e-12
        tried += 1
    P.close()
    assert tried >= 5


@functools.lru_cache(maxsize=1)
def _oracle(grid):
    from oracle import aim, geometry
    from gpu_cases import params_of
    wl = W.SPHERE_L2
    p = params_of(wl)
    s = geometry.Surface(p["xyz"], p["tri"], p["rwg"])
    return s, aim.AIM(s, grid, p["d_near"], p["dt"], wl.f0, p["ng"]), p


@pytest.mark.parametrize("yz", [0, 3])
@pytest.mark.parametrize("grid", [12, (9, 12, 8)], ids=str)
def test_product_plans(grid, yz):
    import torch
    s, A, p = _oracle(grid)
    P = gpu_problem(W.SPHERE_L2.name, nt=8, grid=grid)
    base = dict(P.tuning(), yz_engine=yz)
    m = p["ng"]
    x = W.complex_normal(32, (1, s.ns))
    # the far part by the oracle, the near zone's values (not under test) as exported
    ref = A.far_matvec(m, x[0])
    if m <= P.info["mn"]:
        ref = ref + np.add.reduceat(P.export("near")[m] * x[0][P.export("col")], P.export("rowptr")[:-1])
    xd = torch.from_numpy(x).cuda()
    for a, ax in enumerate("xyz"):
        tried = 0
        for pl in _plans(P.info["padded"][a], 3):
            if not _try(P, dict(base, **{"radix_" + ax: pl})):
                continue
            print("product plans: grid", grid, "engine", yz, "axis", ax, "plan", pl, flush=True)
            assert rel(P.apply_z(m, xd).cpu().numpy()[0], ref) <= 1e-12
            tried += 1
        assert tried >= 3
    P.close()
