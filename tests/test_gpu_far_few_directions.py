"""The far field of up to 8 directions (16 columns: the narrow tile of the
product): rows and columns around the tile's edges (128 rows; two components
per direction, three where one is no unit vector), the first wide product
beside it, and a last direction group that is narrow, against the oracle or the
product of all directions (1e-12, as in the other far-field tests).  And its
time: one direction of 19200 rows once took what 32 take; at most 0.6 of it,
the smallest of ten calls each."""
import time

import pytest

import workloads as W
from gpu_cases import gpu_problem, oracle_aim, rel

pytestmark = pytest.mark.gpu
NAME, TOL = W.SPHERE_L2_NARROW.name, 1e-12


@pytest.mark.parametrize("nd,nt,batch,scale", [(1, 1, 1, 1.0), (2, 16, 1, 1.0), (7, 17, 1, 1.0), (8, 127, 1, 1.0),
                                               (8, 32, 4, 1.0), (8, 43, 3, 1.0), (9, 43, 3, 1.0), (5, 65, 4, 1.25),
                                               (6, 65, 4, 0.5)])
def test_narrow_tile(nd, nt, batch, scale):
    import torch
    from oracle import farfield
    print("few directions:", nd, "steps", nt, "columns", batch, "scale", scale, flush=True)
    s, _, _, p = oracle_aim(NAME)
    dirs = W.unit_vectors(5, 4, nd)
    dirs[-1] *= scale
    F = farfield.FarField(s, dirs, p["dt"], W.SPHERE_L2_NARROW.f0)
    P = gpu_problem(NAME, nt=nt, batch=batch)
    I = W.complex_normal(3, (nt, batch, s.ns))
    U = P.farfield(dirs, torch.from_numpy(I).cuda()).cpu().numpy()
    P.close()
    assert rel(U, F.apply(I)) < TOL


def test_narrow_last_group():
    import torch
    nt, batch = 3, 2
    dirs = W.unit_vectors(6, 4, 1800)
    P = gpu_problem(NAME, nt=nt, batch=batch)
    I = torch.from_numpy(W.complex_normal(7, (nt, batch, P.ns))).cuda()
    ref = torch.cat([P.farfield(dirs[a:a + 600], I) for a in range(0, 1800, 600)], 2)
    # (a group holds a multiple of 32 directions)
    for nd in (1700, 1697, 1729, 1800):
        print("narrow last group: directions", nd, flush=True)
        assert rel(P.farfield(dirs[:nd], I).cpu().numpy(), ref[:, :, :nd].cpu().numpy()) < TOL
    P.close()


def test_one_direction_time():
    import torch
    nt, batch = 300, 64
    P = gpu_problem(W.SPHERE_L2.name, nt=nt, batch=batch)
    I = torch.zeros((nt, batch, P.ns), dtype=torch.complex128, device="cuda")
    best = []
    for nd in (1, 32):
        dirs = W.unit_vectors(5, 4, nd)
        t = []
        for _ in range(12):
            torch.cuda.synchronize()
            a = time.perf_counter()
            P.farfield(dirs, I)
            t.append(time.perf_counter() - a)
        best.append(min(t[2:]))
    P.close()
    print("far field: 1 direction", best[0], "32 directions", best[1], flush=True)
    assert best[0] <= 0.6 * best[1]
