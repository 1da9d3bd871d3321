"""dL/dR of the descriptors where its kernel's partition can go wrong: neighbour
counts around its groups of four (none, one, three to five, the densest cell that
fits), an atom on a grid point, a last tile of one point, at every twojmax,
against the FP64 oracle's chain rule."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 2e-5          # the suite's bound on dL/dR


@pytest.mark.parametrize("tj", [2, 4, 6, 8, 10])
@pytest.mark.parametrize("n_atoms", [0, 1, 3, 4, 5, 9, 120])
def test_neighbour_counts(tj, n_atoms):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    print("twojmax", tj, "atoms", n_atoms, flush=True)
    # a cluster in a large cell, its first atom on a grid point
    L, N, rcut = np.array([30.0, 30.0, 30.0]), np.array([3, 5, 67]), 4.67
    rng = np.random.default_rng(200 * tj + n_atoms)
    v = rng.standard_normal((n_atoms, 3))
    r = 2.2 * rng.random(n_atoms) ** (1 / 3.0)
    pos = np.array([10.0, 12.0, 33 * 30.0 / 67]) + v / np.linalg.norm(v, axis=1, keepdims=True) * r[:, None] \
        if n_atoms else np.zeros((0, 3))
    if n_atoms > 1:
        pos[0] = [10.0, 12.0, 33 * 30.0 / 67]           # the grid's own expression: r = 0 exactly
    snap = mala_synth.Snapshot("cluster", pos, L, N, rcut, tj, 298.0, 1.0)
    n = 961                                             # 15 tiles and one point
    gB = rng.standard_normal((n, oracle.lib().oracle_n_triples(tj))).astype(np.float32)
    ctx = mala.Context(0)
    g = ctx.mala_descriptors_vjp(pos, L, N, rcut, tj, torch.as_tensor(gB, device="cuda"), 0, n)
    ctx.check_device_errors()
    g = g.cpu().numpy()
    ctx.close()
    assert g.shape == (n_atoms, 3) and np.all(np.isfinite(g))
    if n_atoms:
        ref = oracle.descriptors_vjp(snap, gB.astype(np.float64), np.arange(n, dtype=np.int64), nthreads=16)
        err = np.max(np.abs(g - ref)) / np.max(np.abs(ref))
        print("  rel err %.3e" % err, flush=True)
        assert err <= TOL
