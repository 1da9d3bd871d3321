"""FP32 networks whose evening out meets its limits: layers, rows and columns of zeros,
biases far above or below their weights, input and output scales at the ends of the
FP32 range, and slopes outside (0, 1], against the FP64 oracle at the suite's bounds
(1e-5 of a row's largest value, 2e-5 for the vector-Jacobian product; where the outputs
have scales of their own, each counts against its own).  With a slope below zero
sigma(z) has no sign of its own: sigma' goes by the sign of z."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu


def change(net, what, rng):
    W, b = net["W"], net["b"]
    if what == "zero first layer":
        W[0][:] = 0.0
    elif what == "zero rows and columns":
        W[0][3], W[0][:, 5], W[1][7], W[1][:, 9], W[2][11], W[2][:, 2] = 0.0, 0.0, 0.0, 0.0, 0.0, 0.0
        b[0][3] = 0.0
    elif what == "zero biases":
        for v in b:
            v[:] = 0.0
    elif what == "large and small biases":
        b[0][4], b[1][6] = 1e3, -1e3
        W[0][4] *= 1e-6
        b[0][8], b[1][1] = 1e-30, 1e-30
    elif what == "output scales":
        net["out_scale"] = 10.0 ** rng.uniform(-30, 30, len(b[2])) * rng.choice([-1.0, 1.0], len(b[2]))
        net["out_scale"][0] = 0.0
        net["out_shift"] = np.zeros(len(b[2]))
    elif what == "input scales":
        net["in_std"] = 10.0 ** rng.uniform(-12, 12, W[0].shape[1])
        net["in_mean"] = np.zeros(W[0].shape[1])
    elif what.startswith("slope"):
        net["slope"] = float(what.split()[1])
    for x in W + b:
        x[:] = x.astype(np.float32)


@pytest.mark.parametrize("what", ["zero first layer", "zero rows and columns", "zero biases", "large and small biases",
                                  "output scales", "input scales", "slope 0", "slope -0.5", "slope 1.5"])
def test_degenerate(what):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    rng = np.random.default_rng(3)
    net = mala_synth.make_net([30, 64, 80, 50], 4, 8, output_activation=0, egrid=(-5.0, 0.1, 50), with_input_scaler=False)
    change(net, what, rng)
    print(what, flush=True)
    B, v = mala_synth.network_inputs(net, 200, 5)
    ctx = mala.Context(0)
    w = ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32)
    tB = torch.as_tensor(B, device="cuda")
    o = ctx.mala_ldos_infer(w, tB, 50).cpu().double().numpy()
    ref = oracle.mlp(B.astype(np.float64), net, nthreads=16)
    s = np.max(np.abs(ref), axis=0) if what == "output scales" else np.max(np.abs(ref), axis=1, keepdims=True)
    assert np.max(np.abs(o - ref) / np.where(s == 0.0, 1.0, s)) <= 1e-5
    v = (v / np.where(net["out_scale"] == 0.0, 1.0, np.abs(net["out_scale"]))).astype(np.float32)
    g = ctx.mala_ldos_vjp(w, tB, torch.as_tensor(v, device="cuda")).cpu().double().numpy()
    ctx.close()
    gref, margin = oracle.mlp_vjp(B.astype(np.float64), net, v.astype(np.float64), nthreads=16)
    t = np.max(np.abs(gref), axis=0)
    t[t == 0.0] = 1.0
    keep = margin > 1e-5
    if what.startswith("zero"):
        keep[:] = True                               # a unit of zeros has no kink to be near
    rows = np.max(np.abs(gref) / t, axis=1)
    err = np.max(np.abs(g - gref) / t, axis=1) / np.where(rows > 0.0, rows, 1.0)
    assert keep.sum() >= 100 and err[keep].max() <= 2e-5
