"""Networks of at most 128 units in every layer (one unit tile per wave, two blocks per
CU) and those one unit wider, against the FP64 oracle: the LDOS in both precisions,
the vector-Jacobian product, and the whole path, whose reductions run in the same
kernels.  Tolerances are the suite's: 1e-5 of a row's largest value in FP32 and 2e-2
in BF16, 2e-5 for the vector-Jacobian product, and for the whole path DOS 1e-6,
E_F 1e-4 eV, density 1e-5.  The vector-Jacobian product's bound holds for layers of
several units: through a layer of one unit the row is one number times that unit's
weights, a sum whose terms cancel 35,000-fold at the worst of these points (plain
FP32 in numpy is off by 1e-3 there), so that width has its LDOS compared only."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    ctx = mala.Context(0)
    yield mala, ctx, torch
    ctx.close()


def rel(a, b, rows=slice(None)):
    return (np.max(np.abs(a - b), axis=1) / np.max(np.abs(b), axis=1))[rows].max()


@pytest.mark.parametrize("widths", [[128, 128, 128, 128], [128, 128, 129, 128], [91, 113, 128, 129], [17, 16, 127, 3],
                                    [64, 1, 33, 65]])
@pytest.mark.parametrize("n", [1, 63, 65, 16_385, 70_003])
def test_network(env, widths, n):
    mala, ctx, torch = env
    print("widths", widths, "points", n, flush=True)
    net = mala_synth.make_net(widths, sum(widths), 8, egrid=(-5.0, 0.1, widths[-1]), with_input_scaler=False)
    B, v = mala_synth.network_inputs(net, n, 7)
    rows = np.unique(np.linspace(0, n - 1, 600).astype(int))
    tB, tv = torch.as_tensor(B, device="cuda"), torch.as_tensor(v, device="cuda")
    ref = oracle.mlp(B[rows].astype(np.float64), net, nthreads=16)
    blob = mala_synth.net_to_blob(net)
    for prec, tol in ((mala.PREC_FP32, 1e-5), (mala.PREC_BF16, 2e-2)):
        o = ctx.mala_ldos_infer(ctx.weights(blob, prec), tB, widths[-1])
        assert rel(o.cpu().double().numpy()[rows], ref) <= tol
    if min(widths) == 1:
        return
    g = ctx.mala_ldos_vjp(ctx.weights(blob, mala.PREC_FP32), tB, tv).cpu().double().numpy()[rows]
    gref, margin = oracle.mlp_vjp(B[rows].astype(np.float64), net, v[rows].astype(np.float64), nthreads=16)
    keep = (margin > 1e-5) & (np.max(np.abs(gref), axis=1) > 0)
    if keep.any():
        assert rel(g[keep], gref[keep]) <= 2e-5


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n_e", [128, 129])
def test_whole_path(env, n_e, mode):
    mala, ctx, torch = env
    s, eg = mala_synth.with_grid(mala_synth.small(), [20, 21, 19]), (-5.0, 25.0 / n_e, n_e)
    net = mala_synth.make_net([55, 100, 128, n_e], 5, 8, egrid=eg)
    print("energies", n_e, "density mode", mode, flush=True)
    ctx.set_density_mode(mode)
    dos, dens, res = ctx.mala_predict(ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32), s.positions, s.L, s.N, s.rcut,
                                      s.twojmax, eg, s.T, s.n_electrons)
    ctx.check_device_errors()
    ctx.set_density_mode(0)
    ref, r = oracle.predict(s, net, eg), mala.read_result(res)
    assert r["status"] == 0
    assert np.max(np.abs(dos.cpu().numpy() - ref["dos"])) <= 1e-6 * np.max(np.abs(ref["dos"]))
    assert abs(r["e_fermi"] - ref["e_fermi"]) <= 1e-4
    assert np.max(np.abs(dens.cpu().numpy() - ref["density"])) <= 1e-5 * np.max(np.abs(ref["density"]))
