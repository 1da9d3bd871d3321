"""GPU network with FP32 weights as two FP16 planes per operand: widths at the
edges of the unit tiles, of the waves' shares and of the two row forms, point
counts at the edges of the point tiles, and rows whose magnitudes need the
per-point scale, against the FP64 oracle.  The output map is the identity
(scale 1, shift 0, no output activation), so nothing hides the products' error.

Tolerance: a product of two split values is off by at most 2^-22 of itself (the
dropped lo lo and the representation of both), an FP32 sum of k of them by the
rounding of its partial sums; at 512 units and three layers both stay below
1e-6 of the largest output in the mean and 1e-5 (the suite's network bound) at
the worst element."""
import sys

import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    mala.lib()
    ctx = mala.Context(0)
    yield mala, ctx, torch
    ctx.close()


def plain_net(widths, seed):
    net = mala_synth.make_net(widths, seed, 8, output_activation=0, egrid=(-5.0, 0.1, widths[-1]), with_input_scaler=False)
    net["out_scale"] = np.ones(widths[-1])
    net["out_shift"] = np.zeros(widths[-1])
    return net


def infer(env, net, B):
    mala, ctx, torch = env
    print("widths", net["widths"], "points", len(B), flush=True)
    sys.stdout.flush()
    w = ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32)
    out = ctx.mala_ldos_infer(w, torch.as_tensor(B, device="cuda"), net["widths"][-1])
    ctx.synchronize()
    return out.cpu().double().numpy()


def rel_rows(a, b):
    return np.max(np.abs(a - b), axis=1) / np.maximum(np.max(np.abs(b), axis=1), 1e-300)


@pytest.mark.parametrize("widths,n", [([1, 1, 1, 2], 1), ([16, 16, 17, 16], 31), ([17, 127, 129, 250], 33), ([64, 384, 400, 256], 64),
                                      ([65, 385, 399, 3], 65), ([91, 400, 401, 250], 129), ([128, 512, 496, 256], 97),
                                      ([55, 137, 33, 121], 8193), ([91, 280, 264, 250], 256 * 64 + 1)])
def test_widths_and_point_counts(env, widths, n):
    net = plain_net(widths, sum(widths))
    rng = np.random.default_rng(n)
    B = rng.standard_normal((n, widths[0])).astype(np.float32)
    err = rel_rows(infer(env, net, B), oracle.mlp(B.astype(np.float64), net, nthreads=16))
    print("  rel err %.3e" % err.max(), flush=True)
    assert err.max() <= TOL


def test_rows_of_any_magnitude_and_not_finite(env):
    """Each point has its own scale: rows of 1e-30 to 1e30 side by side, a zero
    row, and rows with NaN or an infinity, which stay in their own rows."""
    net = plain_net([91, 400, 400, 250], 5)
    for b in net["b"]:
        b[:] = 0.0                                    # the output scales with the row
    rng = np.random.default_rng(7)
    B = (rng.standard_normal((200, 91)) * 10.0 ** rng.integers(-30, 31, (200, 1))).astype(np.float32)
    B[3] = 0.0
    B[3, 5] = 1e-38
    ref = oracle.mlp(B.astype(np.float64), net, nthreads=16)
    clean = infer(env, net, B)
    assert rel_rows(clean, ref)[np.arange(200) != 3].max() <= TOL
    B[10, 4], B[70, 90], B[130, 0] = np.nan, np.inf, -np.inf
    out = infer(env, net, B)
    bad = [10, 70, 130]
    assert np.all(~np.isfinite(out[bad]).any(axis=1))
    keep = np.setdiff1d(np.arange(200), bad)
    assert np.array_equal(out[keep], clean[keep])


def test_weights_of_any_magnitude(env):
    """Each layer has its own scale: weights of 1e-20 and of 1e20."""
    net = plain_net([55, 100, 100, 64], 9)
    for W, b, f in zip(net["W"], net["b"], (1e-20, 1e20, 1e-3)):
        W *= f
        b[:] = 0.0
        W[:] = W.astype(np.float32)
    B = np.random.default_rng(1).standard_normal((77, 55)).astype(np.float32)
    err = rel_rows(infer(env, net, B), oracle.mlp(B.astype(np.float64), net, nthreads=16))
    assert err.max() <= TOL
