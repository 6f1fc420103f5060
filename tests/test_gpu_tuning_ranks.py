"""The autotuner on a grid whose product does not depend on the radix plans and
the y/z engine (register x lines and the plane kernel, 18^3): what no launch
takes stays as it was, and the y/z engine and plans, which the commit and the
delayed field still take, are not slower there than the defaults.  A delayed
field call holds N_g commits and one history sum; the bound of 1.15 on the
smallest of 15 calls each leaves room for the clock."""
import pytest

import workloads as W
from gpu_cases import gpu_problem

pytestmark = pytest.mark.gpu


def _ms(P, torch, hist):
    best = 1e9
    for _ in range(15):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        P.delayed_field(hist)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("precision,batch", [(0, 1), (1, 8)])
def test_plans_of_the_history(precision, batch):
    import torch
    P = gpu_problem(W.SPHERE_L3.name, precision=precision, batch=batch, nt=8, tol=1e-4)
    base = P.tuning()
    hist = torch.from_numpy(W.complex_normal(3, (P.info["ng"], batch, P.ns))).cuda()
    t = P.autotune(budget_ms=4000)
    print("tuned", t, flush=True)
    for f in ("radix_x", "gather_rows", "lines_per_block"):
        assert t[f] == base[f], f
    tuned = _ms(P, torch, hist)
    keep = {f: base[f] for f in ("radix_y", "radix_z", "yz_engine", "delay_block")}
    P.set_tuning(dict(t, **keep))
    default = _ms(P, torch, hist)
    print("history", precision, batch, "tuned", tuned, "default", default, flush=True)
    assert tuned <= 1.15 * default
    P.close()
