"""FP32 network where magnitudes spread inside a layer: inputs, hidden units and
outputs scaled over many decades with the scale taken back by the next layer (the
same function, which FP32 computes with the same error), a large input that no unit
reads, and two halves of a network, one 1e8 times the other, that never meet
(nothing can even those out, so the operands' own range has to hold them), for the
LDOS and the vector-Jacobian product, against the FP64 oracle.

Tolerances: the network's own (1e-5 of the largest output of a row at worst, 2e-5 of
the largest component for the vector-Jacobian product).  In the 2-norm: three layers,
each a sum of k <= 400 products whose partial sums round to 2^-24 (0.6 of that
in the mean, sqrt(k / 32) of them of a size that matters) and operands good to 2^-23:
below 1e-6."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL, TOL_VJP, TOL_NORM, MARGIN = 1e-5, 2e-5, 1e-6, 1e-5


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    ctx = mala.Context(0)
    yield mala, ctx, torch
    ctx.close()


def plain_net(widths, seed):
    net = mala_synth.make_net(widths, seed, 8, output_activation=0, egrid=(-5.0, 0.1, widths[-1]), with_input_scaler=False)
    net["out_scale"], net["out_shift"] = np.ones(widths[-1]), np.zeros(widths[-1])
    return net


def rounded(net):
    net["W"] = [W.astype(np.float32).astype(np.float64) for W in net["W"]]
    net["b"] = [b.astype(np.float32).astype(np.float64) for b in net["b"]]
    return net


def check(env, net, B, v, outputs=None):
    """outputs: scale of each output, against which its error counts."""
    mala, ctx, torch = env
    w = ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32)
    print("widths", net["widths"], "points", len(B), flush=True)
    o = ctx.mala_ldos_infer(w, torch.as_tensor(B, device="cuda"), net["widths"][-1]).cpu().double().numpy()
    ref = oracle.mlp(B.astype(np.float64), net, nthreads=16)
    s = np.ones(ref.shape[1]) if outputs is None else outputs
    err = np.max(np.abs(o - ref) / s, axis=1) / np.max(np.abs(ref) / s, axis=1)
    norm = np.linalg.norm((o - ref) / s) / np.linalg.norm(ref / s)
    g = ctx.mala_ldos_vjp(w, torch.as_tensor(B, device="cuda"), torch.as_tensor(v, device="cuda")).cpu().double().numpy()
    gref, margin = oracle.mlp_vjp(B.astype(np.float64), net, v.astype(np.float64), nthreads=16)
    t = np.max(np.abs(gref), axis=0)                 # a component's own scale
    t[t == 0.0] = 1.0
    gerr = (np.max(np.abs(g - gref) / t, axis=1) / np.max(np.abs(gref) / t, axis=1))[margin > MARGIN]
    print("  ldos max %.2e norm %.2e  vjp max %.2e (%d points)" % (err.max(), norm, gerr.max(), len(gerr)), flush=True)
    assert len(gerr) >= 0.8 * len(B)
    assert err.max() <= TOL and norm <= TOL_NORM and gerr.max() <= TOL_VJP


@pytest.mark.parametrize("widths", [[91, 400, 400, 250], [55, 100, 180, 121]])
@pytest.mark.parametrize("decades", [0, 8, 14])
def test_scales_taken_back(env, widths, decades):
    net = plain_net(widths, sum(widths))
    rng = np.random.default_rng(decades + widths[0])
    B = rng.standard_normal((200, widths[0])).astype(np.float32)
    v = rng.standard_normal((200, widths[-1])).astype(np.float32)
    check(env, net, B, v)
    s = [10.0 ** rng.uniform(-decades / 2, decades / 2, w) for w in widths]
    W, b = net["W"], net["b"]
    for l in range(3):                               # unit i of layer l + 1 times s[l + 1][i]
        net = dict(net)
        net["W"] = [W[m] * (s[m + 1][:, None] if m <= l else 1.0) / (s[m][None, :] if m <= l else 1.0) for m in range(3)]
        if l < 2:
            net["W"][l + 1] = net["W"][l + 1] / s[l + 1][None, :]
        net["b"] = [b[m] * (s[m + 1] if m <= l else 1.0) for m in range(3)]
        check(env, rounded(net), (B * s[0]).astype(np.float32), (v / s[3] if l == 2 else v).astype(np.float32),
              s[3] if l == 2 else None)


def test_large_input_that_nothing_reads(env):
    net = plain_net([91, 400, 400, 250], 3)
    net["W"][0][:, [7, 90]] = 0.0
    rng = np.random.default_rng(4)
    B = rng.standard_normal((200, 91))
    B[:, [7, 90]] *= 1e12
    check(env, net, B.astype(np.float32), rng.standard_normal((200, 250)).astype(np.float32))


@pytest.mark.parametrize("widths", [[90, 400, 400, 250], [54, 100, 180, 120]])
def test_halves_that_never_meet(env, widths):
    net = plain_net(widths, 11)
    half = [w // 2 for w in widths]
    for l in range(3):
        net["W"][l][:half[l + 1], half[l]:] = 0.0
        net["W"][l][half[l + 1]:, :half[l]] = 0.0
        net["b"][l][:] = 0.0
    rng = np.random.default_rng(12)
    B, v = rng.standard_normal((200, widths[0])), rng.standard_normal((200, widths[-1]))
    B[:, half[0]:] *= 1e8
    s = np.where(np.arange(widths[-1]) < half[-1], 1.0, 1e8)
    check(env, net, B.astype(np.float32), v.astype(np.float32), s)
    v[:, :half[-1]] *= 1e-8                          # the vector's spread goes the other way
    check(env, net, B.astype(np.float32), v.astype(np.float32), s)
