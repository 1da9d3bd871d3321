"""Angle and cutoff phase per unit distance keep their precision: at cutoffs where
0.99363 pi / rcut, formed and held in one float, would be off by up to 1.3e-7, the
descriptors and their gradient have no error that all neighbours share.  Such an
error is the one of a slightly different cutoff, so it is measured as the part of the
error along the derivative with respect to ln rcut (FP64 oracle, central difference,
a neighbour on the cutoff sphere contributing nothing to first order); what a float
rounds at random averages out over the points.

Tolerance: the two floats hold the factor to 2^-48.  A descriptor row's random error
is about 3e-7 of the row and the derivative of order 1 to 10 of it, so over 800 rows
the random part is below 3e-7 / sqrt(800) = 1e-8; a gradient's error is 1e-6 over 96
components whose derivative is of order 1 to 10, 1e-6 / sqrt(96) / 3 = 3e-8."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu


def along(err, derivative):
    return float(np.sum(err * derivative) / np.sum(derivative * derivative))


@pytest.mark.parametrize("rcut", [4.4275, 4.3127, 4.2021])
def test_no_common_error(rcut):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    s, tj, h = mala_synth.small(), 10, 1e-3
    pts = np.arange(2000, 2800, dtype=np.int64)
    at = lambda r: mala_synth.Snapshot(s.name, s.positions, s.L, s.N, r, tj, s.T, s.n_electrons)
    ctx = mala.Context(0)
    B = ctx.mala_descriptors(s.positions, s.L, s.N, rcut, tj, 2000, 2800).cpu().double().numpy()
    ref, up, down = (oracle.descriptors(at(r), pts, nthreads=16) for r in (rcut, rcut * (1 + h), rcut * (1 - h)))
    scale = np.max(np.abs(ref), axis=1, keepdims=True)
    e = along((B - ref) / scale, (up - down) / (2 * h) / scale)
    gB = np.random.default_rng(1).standard_normal(ref.shape).astype(np.float32)
    g = ctx.mala_descriptors_vjp(s.positions, s.L, s.N, rcut, tj, torch.as_tensor(gB, device="cuda"), 2000, 2800)
    gref, gup, gdown = (oracle.descriptors_vjp(at(r), gB.astype(np.float64), pts, nthreads=16)
                        for r in (rcut, rcut * (1 + h), rcut * (1 - h)))
    eg = along(g.cpu().numpy() - gref, (gup - gdown) / (2 * h))
    ctx.check_device_errors()
    ctx.close()
    print("rcut %g: common error %.2e of the descriptors, %.2e of the gradient" % (rcut, e, eg), flush=True)
    assert abs(e) <= 1e-8 and abs(eg) <= 3e-8
