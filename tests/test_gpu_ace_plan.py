"""Grid ACE descriptors (ranks 1-3, and rank 4) over every basis size their plans
are built for, point-major and descriptor-major, at point counts around the
kernels' 8-, 16- and 64-point tiles and into outputs that are and are not 16-byte
aligned, against the FP64 oracle."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5          # the suite's bound on a descriptor row


def check(nd, call, ref, counts):
    import torch
    for n in counts:
        for planes in (False, True):
            for shift in (0, 1):
                print("points", n, "planes", planes, "shift", shift, flush=True)
                buf = torch.full((n * nd + 2,), 7.5, dtype=torch.float32, device="cuda")
                out = buf[shift:shift + n * nd].view((nd, n) if planes else (n, nd))
                call(n, out, planes)
                g = (out.T if planes else out).cpu().double().numpy()
                err = np.max(np.max(np.abs(g - ref[:n]), axis=1) / np.max(np.abs(ref[:n]), axis=1))
                assert err <= TOL, err
                # nothing beside the rows is written
                assert float(buf[shift + n * nd]) == 7.5 and (shift == 0 or float(buf[0]) == 7.5)


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    ctx = mala.Context(0)
    yield mala, ctx
    ctx.close()


@pytest.mark.parametrize("nmax", [1, 2, 3, 4])
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 4])
def test_ranks123(env, nmax, lmax):
    mala, ctx = env
    s, begin = mala_synth.small(), 1000
    ref = oracle.ace(s, s.rcut, nmax, lmax, np.arange(begin, begin + 129, dtype=np.int64), nthreads=16)

    def call(n, out, planes):
        ctx.mala_ace_descriptors(s.positions, s.L, s.N, s.rcut, nmax, lmax, begin, begin + n, out=out,
                                 descriptor_major=planes)
        ctx.check_device_errors()
    check(mala.ace_count(nmax, lmax), call, ref, (1, 15, 16, 17, 64, 129))


@pytest.mark.parametrize("nmax4", [1, 2, 3])
@pytest.mark.parametrize("lmax4", [0, 1, 2, 3])
def test_rank4(env, nmax4, lmax4):
    mala, ctx = env
    s, begin = mala_synth.small(), 1000
    ref = oracle.ace4(s, s.rcut, nmax4, lmax4, np.arange(begin, begin + 129, dtype=np.int64), nthreads=16)

    def call(n, out, planes):
        ctx.mala_ace4_descriptors(s.positions, s.L, s.N, s.rcut, nmax4, lmax4, begin, begin + n, out=out,
                                  descriptor_major=planes)
        ctx.check_device_errors()
    check(mala.ace4_count(nmax4, lmax4), call, ref, (1, 7, 8, 9, 64, 129))
