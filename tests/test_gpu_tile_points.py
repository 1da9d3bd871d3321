"""Points and boxes of the neighbour kernels' tiles over grids whose 64-point tiles
cross rows, planes and several planes, from ranges that start inside them, against
the FP64 oracle."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5          # the suite's bound on a descriptor row


@pytest.mark.parametrize("N", [(3, 5, 67), (40, 7, 3), (64, 2, 2), (9, 11, 64), (1, 1, 300), (200, 3, 1), (7, 1, 129),
                               (300, 1, 1), (5, 20, 63)])
def test_grids(N):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    L, tj = np.array([8.1, 9.0, 10.2]), 2
    pos = np.random.default_rng(sum(N)).random((40, 3)) * L
    snap = mala_synth.Snapshot("grid", pos, L, np.array(N), 4.67, tj, 298.0, 1.0)
    total = int(np.prod(N))
    ctx = mala.Context(0)
    for begin in (0, 13, total // 2):
        print("grid", N, "from", begin, flush=True)
        B = ctx.mala_descriptors(pos, L, np.array(N), 4.67, tj, begin, total).cpu().double().numpy()
        ctx.check_device_errors()
        ref = oracle.descriptors(snap, np.arange(begin, total, dtype=np.int64), nthreads=16)
        err = np.max(np.abs(B - ref), axis=1) / np.max(np.abs(ref), axis=1)
        print("  rel err %.3e" % err.max(), flush=True)
        assert err.max() <= TOL
    ctx.close()
