"""FP32 network and its vector-Jacobian product for points with an infinite input, an
activation that overflows, or an infinite vector: where plain FP32 has an infinity
or a finite value, so have they.  The gradient of a point with an infinite input is
finite: its units' signs are those of the infinities of the first layer, and
sigma' is the slope where the second layer is not a number.  Reference: the same
formulas in numpy, 64 bits.  Widths at multiples of a tile and not, an infinity in
the first, an inner and the last input (whose column is read for the padding)."""
import numpy as np
import pytest

import mala_synth

pytestmark = pytest.mark.gpu

TOL, TOL_VJP = 1e-5, 2e-5          # the suite's bounds for the network and its vector-Jacobian product


def reference(net, B, v):
    W, b, slope = net["W"], net["b"], net["slope"]
    with np.errstate(all="ignore"):
        act = lambda z: np.where(z < 0, slope * z, z)
        mask = lambda h: np.where(h > 0, 1.0, slope)
        x = (B.astype(np.float64) - net["in_mean"]) / net["in_std"]
        h1 = act(x @ W[0].T + b[0])
        h2 = act(h1 @ W[1].T + b[1])
        y = h2 @ W[2].T + b[2]
        d = v * net["out_scale"]
        if net["output_activation"]:
            d = d * mask(y)
            y = act(y)
        g = ((d @ W[2] * mask(h2)) @ W[1] * mask(h1)) @ W[0] / net["in_std"]
        return y * net["out_scale"] + net["out_shift"], g


def same(a, ref, tol, rows):
    a, ref = a[rows], ref[rows]
    big = np.abs(ref) > 3.4e38                       # an overflow in FP32
    finite = np.isfinite(ref) & ~big
    assert np.array_equal(np.isnan(a), np.isnan(ref))
    assert np.array_equal(np.sign(a[~finite & ~np.isnan(ref)]), np.sign(ref[~finite & ~np.isnan(ref)]))
    assert np.isinf(a[~finite & ~np.isnan(ref)]).all()
    for r in range(len(a)):
        f = finite[r]
        if f.any():
            assert np.max(np.abs(a[r, f] - ref[r, f])) <= tol * np.max(np.abs(ref[r, f])), r


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    ctx = mala.Context(0)
    yield mala, ctx, torch
    ctx.close()


def run(env, net, B, v, vjp=True):
    mala, ctx, torch = env
    print("widths", net["widths"], "points", len(B), flush=True)
    w = ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32)
    tB, tv = torch.as_tensor(B, device="cuda"), torch.as_tensor(v, device="cuda")
    o = ctx.mala_ldos_infer(w, tB, net["widths"][-1]).cpu().double().numpy()
    return o, ctx.mala_ldos_vjp(w, tB, tv).cpu().double().numpy() if vjp else None


@pytest.mark.parametrize("widths", [[91, 400, 400, 250], [55, 100, 110, 250], [80, 160, 432, 256]])
@pytest.mark.parametrize("n", [97, 20_000])
def test_infinite_inputs(env, widths, n):
    net = mala_synth.make_net(widths, 3, 8, egrid=(-5.0, 0.1, widths[-1]), with_input_scaler=False)
    B, v = mala_synth.network_inputs(net, n, 5)
    clean_o, clean_g = run(env, net, B, v)
    bad = [0, 40, 63, n - 1]
    B[0, 0], B[40, widths[0] - 1], B[63, widths[0] // 2], B[n - 1, 3] = np.inf, -np.inf, np.inf, -np.inf
    o, g = run(env, net, B, v)
    keep = np.setdiff1d(np.arange(n), bad)
    assert np.array_equal(o[keep], clean_o[keep]) and np.array_equal(g[keep], clean_g[keep])
    ro, rg = reference(net, B[bad], v[bad])
    assert np.isfinite(rg).all()
    same(o[bad], ro, TOL, slice(None))
    same(g[bad], rg, TOL_VJP, slice(None))


def test_overflow_and_infinite_vector(env):
    # one unit of the second layer overflows; and a vector with one infinity
    net = mala_synth.make_net([16, 32, 48, 64], 3, 8, output_activation=0, egrid=(-5.0, 0.1, 64), with_input_scaler=False)
    net["W"][1][5] = np.float32(1e38)
    net["out_scale"], net["out_shift"] = np.ones(64), np.zeros(64)
    rng = np.random.default_rng(2)
    B = np.abs(rng.standard_normal((70, 16))).astype(np.float32) * 10
    net["W"][0] = np.abs(net["W"][0])                # positive units: the sum overflows upwards
    o, _ = run(env, net, B, np.zeros((70, 64), np.float32))
    assert np.isinf(o).all() and np.array_equal(np.sign(o), np.broadcast_to(np.sign(net["W"][2][:, 5]), o.shape))
    net["W"][1][5] = 0.1
    v = rng.standard_normal((70, 64)).astype(np.float32)
    _, clean = run(env, net, B, v)
    v[11, 4] = np.inf
    _, g = run(env, net, B, v)
    same(g[[11]], reference(net, B[[11]], v[[11]])[1], TOL_VJP, slice(None))
    assert np.array_equal(np.delete(g, 11, 0), np.delete(clean, 11, 0))
