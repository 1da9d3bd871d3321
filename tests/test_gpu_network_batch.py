"""A point's values do not depend on how many points are in the call: the network
and its vector-Jacobian product over a range of rows give the bits of the same
rows among many, at hidden widths whose unit tiles leave every remainder over the
eight waves (the leftover tiles are computed one way or the other by the point
tiles of a block, and those follow the number of points), in both precisions."""
import pytest

import mala_synth

pytestmark = pytest.mark.gpu

N = 40_000          # 64-point tiles on every block (96-point ones for BF16)
RANGES = [(0, 1), (0, 100), (31, 64), (12_345, 20_345), (39_967, 40_000)]


@pytest.mark.parametrize("h1,h2", [(176, 176), (304, 432), (432, 304), (400, 150), (64, 200), (500, 270)])
def test_same_bits_in_small_and_large_calls(h1, h2):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    net = mala_synth.make_net([91, h1, h2, 250], h1 + h2, 10)
    B, v = (torch.as_tensor(a, device="cuda") for a in mala_synth.network_inputs(net, N, 3))
    ctx = mala.Context(0)
    blob = mala_synth.net_to_blob(net)
    w32, w16 = ctx.weights(blob, mala.PREC_FP32), ctx.weights(blob, mala.PREC_BF16)
    calls = {"fp32": lambda s: ctx.mala_ldos_infer(w32, B[s], 250), "bf16": lambda s: ctx.mala_ldos_infer(w16, B[s], 250)}
    if h1 + h2 < 770:                            # wider ones are refused
        calls["vjp"] = lambda s: ctx.mala_ldos_vjp(w32, B[s], v[s])
    for name, call in calls.items():
        print("widths", h1, h2, name, flush=True)
        whole = call(slice(0, N))
        for a, b in RANGES:
            assert torch.equal(call(slice(a, b)), whole[a:b]), (a, b)
    ctx.close()
