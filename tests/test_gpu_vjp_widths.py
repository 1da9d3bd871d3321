"""Widths that the network's vector-Jacobian product accepts and refuses: both hidden
layers and the wider of input and output, each rounded up to 64 units, of at most 1152
together.  Accepted ones are compared with the FP64 oracle at the suite's bound."""
import numpy as np
import pytest

import mala_synth
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,ok", [([91, 448, 448, 256], True), ([91, 448, 449, 256], False), ([128, 512, 512, 128], True),
                                       ([128, 512, 512, 129], False), ([91, 512, 384, 250], True), ([91, 512, 400, 250], False),
                                       ([1, 385, 512, 193], False), ([33, 385, 448, 193], True), ([91, 400, 400, 250], True)])
def test_widths(widths, ok):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    print("widths", widths, flush=True)
    net = mala_synth.make_net(widths, sum(widths), 8, egrid=(-5.0, 0.1, widths[-1]), with_input_scaler=False)
    B, v = mala_synth.network_inputs(net, 300, 9)
    ctx = mala.Context(0)
    w = ctx.weights(mala_synth.net_to_blob(net), mala.PREC_FP32)
    call = lambda: ctx.mala_ldos_vjp(w, torch.as_tensor(B, device="cuda"), torch.as_tensor(v, device="cuda"))
    if not ok:
        with pytest.raises(mala.MalaError, match="1152"):
            call()
    else:
        g = call().cpu().double().numpy()
        ref, margin = oracle.mlp_vjp(B.astype(np.float64), net, v.astype(np.float64), nthreads=16)
        err = np.max(np.abs(g - ref), axis=1) / np.max(np.abs(ref), axis=1)
        assert (margin > 1e-5).sum() >= 0.8 * len(B) and err[margin > 1e-5].max() <= 2e-5
    ctx.close()
