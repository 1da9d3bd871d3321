"""Cell list by one block and by the general path: atom and cell counts on both
sides of the line between them, atoms outside the cell (wrapped) and on its faces,
against the FP64 oracle's descriptors, which search all images."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5          # the suite's bound on a descriptor row


# atoms, cell edge (16 cells of rcut/2 per edge below 39.695, 17 from there on)
@pytest.mark.parametrize("n_atoms,edge", [(0, 12.0), (1, 5.0), (1025, 24.0), (4096, 37.5), (4097, 37.5), (4096, 39.8),
                                          (300, 39.8)])
def test_paths(n_atoms, edge):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    print("atoms", n_atoms, "edge", edge, flush=True)
    rng = np.random.default_rng(n_atoms + int(10 * edge))
    pos = (rng.random((n_atoms, 3)) * 3.0 - 1.0) * edge
    if n_atoms > 3:
        pos[0], pos[1], pos[2] = 0.0, edge, -edge
    L, N, tj = np.array([edge] * 3), np.array([9, 11, 40]), 4
    snap = mala_synth.Snapshot("box", pos, L, N, 4.67, tj, 298.0, 1.0)
    ctx = mala.Context(0)
    B = ctx.mala_descriptors(pos, L, N, 4.67, tj, 100, 100 + 333).cpu().double().numpy()
    ctx.check_device_errors()
    ctx.close()
    ref = oracle.descriptors(snap, np.arange(100, 433, dtype=np.int64), nthreads=16)
    err = np.max(np.abs(B - ref), axis=1) / np.max(np.abs(ref), axis=1)
    print("  rel err %.3e" % err.max(), flush=True)
    assert err.max() <= TOL
