"""Device arrays shorter than a call reads or writes: a time series that ends
early (excitation, adjoint source, currents, far field) continues with zeros,
as if the zeros had been passed; anything else that is too short is refused
before an address reaches a kernel."""
import numpy as np
import pytest

import workloads as W
from gpu_cases import gpu_problem

pytestmark = pytest.mark.gpu


def _zeros_after(t, steps):
    import torch
    out = torch.zeros((steps,) + tuple(t.shape[1:]), dtype=t.dtype, device=t.device)
    out[:len(t)] = t
    return out


def test_series_that_end_early():
    import torch
    nt, batch, dirs = 8, 2, W.unit_vectors(5, 4, 3)
    P = gpu_problem(W.SPHERE_L2.name, nt=nt, batch=batch, tol=1e-8)
    V = torch.from_numpy(W.complex_normal(3, (3, batch, P.ns))).cuda()
    Ub = torch.from_numpy(W.complex_normal(4, (3, batch, 3, 3))).cuda()
    full = _zeros_after(V, nt)
    I = P.march(full)[0]
    assert torch.equal(P.march(V)[0], I)
    assert torch.equal(P.march(V, nsteps=3)[0][:3], I[:3])
    part = P.march(full, nsteps=5)[0]
    assert torch.equal(P.march_continue(V, part, 5, 3)[0], I)
    assert torch.equal(P.adjoint_march(V)[0], P.adjoint_march(full)[0])
    assert torch.equal(P.farfield(dirs, V), P.farfield(dirs, full))
    assert torch.equal(P.farfield_adjoint(dirs, Ub), P.farfield_adjoint(dirs, _zeros_after(Ub, nt)))
    P.close()


def test_short_arrays_are_refused():
    import torch
    nt, batch, dirs = 8, 2, W.unit_vectors(5, 4, 3)
    P = gpu_problem(W.SPHERE_L2.name, nt=nt, batch=batch, tol=1e-8)

    def z(*shape, dtype=torch.complex128):
        return torch.zeros(shape, dtype=dtype, device="cuda")
    V, k = z(nt, batch, P.ns), W.unit_vectors(2, 2, batch)
    for call in (lambda: P.march(V, out=z(nt - 1, batch, P.ns)),
                 lambda: P.march(V, out=z(2, batch, P.ns), nsteps=3),
                 lambda: P.march(V.to(torch.complex64)),
                 lambda: P.apply_z(0, z(1, P.ns)),
                 lambda: P.delayed_field(z(P.info["ng"] - 1, batch, P.ns)),
                 lambda: P.excitation(k, W.polarisations(2, k), 1e-8, 1e-7, out=z(nt - 1, batch, P.ns)),
                 lambda: P.excitation(k, W.polarisations(2, k)[:1], 1e-8, 1e-7),
                 lambda: P.farfield(dirs[:, :2], V),
                 lambda: P.rcs(z(nt, batch, 2, 3), np.eye(3), [0.0], 1e-8)):
        with pytest.raises(ValueError):
            call()
    I = P.march(V, nsteps=3)[0]
    with pytest.raises(ValueError):
        P.march_continue(V, I[:4].contiguous(), 3, 2)
    P.close()
