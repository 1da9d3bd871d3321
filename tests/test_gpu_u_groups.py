"""Expansion sums of the descriptor kernel where its partition can go wrong:
neighbour counts around its chunks of eight and lists filled by all four waves
(no neighbour, one, seven to nine, the densest cell that fits), at every
twojmax, against the FP64 oracle."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5          # the suite's bound on a descriptor row


@pytest.mark.parametrize("tj", [2, 4, 6, 8, 10])
@pytest.mark.parametrize("n_atoms", [0, 1, 7, 8, 9, 17, 120])
def test_neighbour_counts(tj, n_atoms):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    print("twojmax", tj, "atoms", n_atoms, flush=True)
    # every atom within the cutoff of the grid's points: a cluster in a large cell
    L, N, rcut = np.array([30.0, 30.0, 30.0]), np.array([3, 5, 67]), 4.67
    rng = np.random.default_rng(100 * tj + n_atoms)
    v = rng.standard_normal((n_atoms, 3))
    r = 2.2 * rng.random(n_atoms) ** (1 / 3.0)
    pos = 15.0 + v / np.linalg.norm(v, axis=1, keepdims=True) * r[:, None] if n_atoms else np.zeros((0, 3))
    snap = mala_synth.Snapshot("cluster", pos, L, N, rcut, tj, 298.0, 1.0)
    pts = np.arange(snap.n_points, dtype=np.int64)
    ctx = mala.Context(0)
    B = ctx.mala_descriptors(pos, L, N, rcut, tj).cpu().double().numpy()
    ctx.check_device_errors()
    ref = oracle.descriptors(snap, pts, nthreads=16)
    err = np.max(np.abs(B - ref), axis=1) / np.max(np.abs(ref), axis=1)
    print("  rel err %.3e" % err.max(), flush=True)
    assert err.max() <= TOL
    ctx.close()
