"""The far field's work space counts in device_bytes while the context keeps
it, and no longer once a call too large to keep it has freed it."""
import pytest

import workloads as W
from gpu_cases import gpu_problem

pytestmark = pytest.mark.gpu


def test_work_space_is_counted():
    import torch
    print("far field: device_bytes", flush=True)
    nt, batch = 210, 100
    P = gpu_problem(W.SPHERE_L2_NARROW.name, nt=nt, batch=batch)
    before = P.describe()["device_bytes"]
    I = torch.zeros((nt, batch, P.ns), dtype=torch.complex128, device="cuda")
    U = P.farfield(W.unit_vectors(5, 4, 2), I)
    # the basis functions' tap table alone: two directions, two components, five taps and more
    kept = P.describe()["device_bytes"] - before
    assert kept >= 2 * 2 * 5 * P.ns * 16
    P.farfield(W.unit_vectors(5, 4, 2), I)
    assert P.describe()["device_bytes"] - before == kept
    P.farfield_adjoint(W.unit_vectors(5, 4, 2), U)
    assert P.describe()["device_bytes"] - before >= kept
    # 500 directions of 21000 rows: 336 MB of products, freed at the end of the call
    P.farfield(W.unit_vectors(5, 4, 500), I)
    assert P.describe()["device_bytes"] == before
    P.close()
