"""Reductions of a stored LDOS at the edges of their partition (fewer points than
partial rows, than row groups, than the four points a wave takes; odd energy
counts) against the FP64 oracle on identical input."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# FP64 sums of float32 values in another order: a few ulp per term, far below
TOL = 1e-12


@pytest.mark.parametrize("n,ne", [(1, 2), (2, 63), (3, 64), (5, 65), (511, 250), (513, 255), (2049, 256), (33_001, 250), (70_003, 129)])
def test_integrate_partition_edges(n, ne):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    print("points", n, "energies", ne, flush=True)
    eg, T, dV = (-5.0, 25.0 / ne, ne), 700.0, 0.01
    rng = np.random.default_rng(n + ne)
    ld = (0.05 + 0.1 * rng.random((n, ne))).astype(np.float32)
    D = oracle.dos(ld.astype(np.float64), dV)
    e = eg[1] * np.sum(0.5 * (D[1:] + D[:-1]))
    target = 0.6 * e                                   # reached inside the grid
    ctx = mala.Context(0)
    dos, dens, res = ctx.mala_integrate(torch.as_tensor(ld, device="cuda"), dV, eg, T, target)
    r = mala.read_result(res)
    ref = oracle.fermi(D, eg, T, target)
    assert r["status"] == mala.MALA_OK
    assert np.max(np.abs(dos.cpu().numpy() - D)) <= TOL * np.max(np.abs(D))
    assert abs(r["e_fermi"] - ref["e_fermi"]) <= 1e-10
    n_ref = oracle.density(ld.astype(np.float64), ref["weights"])
    assert np.max(np.abs(dens.cpu().numpy() - n_ref)) <= 1e-9 * np.max(np.abs(n_ref))
    ctx.close()
