"""Grid ACE calls in either layout can be captured into a graph once a call of the
same size has been made in one of them: that first call makes everything a later one
needs.  The graph is replayed several times, with eager work between, and each
replay compared with the eager result."""
import pytest

import mala_synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [False, True])
@pytest.mark.parametrize("rank4", [False, True])
def test_other_layout_under_capture(rank4, first):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    s, n = mala_synth.small(), 1000
    ctx = mala.Context(0)
    call = ctx.mala_ace4_descriptors if rank4 else ctx.mala_ace_descriptors
    print("rank 4" if rank4 else "ranks 1-3", "first layout", int(first), flush=True)
    run = lambda dm, out=None: call(s.positions, s.L, s.N, s.rcut, 3, 3, 0, n, out=out, descriptor_major=dm)
    run(first)
    out = torch.zeros(run(first).T.shape, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(not first, out)
    fresh = mala.Context(0)
    ref = (fresh.mala_ace4_descriptors if rank4 else fresh.mala_ace_descriptors)(
        s.positions, s.L, s.N, s.rcut, 3, 3, 0, n, descriptor_major=not first)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    ctx.close()
    fresh.close()
