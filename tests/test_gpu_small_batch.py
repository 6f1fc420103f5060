"""Products around the edges of the small-batch kernels: the anterpolation by
lane groups (up to two columns, or few sums) and by lanes, and the
interpolation for one, up to four and up to 32 columns per wave, whose last
pass holds a remainder.  Z_0 (near-zone values of their own array), a lag
inside and one outside the near zone, against the oracle: 1e-12 in FP64 as
the other operator tests, 1e-5 in FP32."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim, oracle_matvec, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 33])
def test_products(batch, precision, tol):
    import torch
    name = W.SPHERE_L2.name
    print("products: columns", batch, "precision", precision, flush=True)
    s, A, _, p = oracle_aim(name)
    P = gpu_problem(name, precision=precision, batch=batch)
    x = W.complex_normal(batch, (batch, s.ns))
    cols = sorted({0, batch // 2, batch - 1})
    for m in (0, 1, p["ng"]):
        y = P.apply_z(m, torch.from_numpy(x).cuda()).cpu().numpy()
        assert rel(y[cols], oracle_matvec(name, m, x[cols])) <= tol
    P.close()
