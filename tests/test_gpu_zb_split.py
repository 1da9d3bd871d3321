"""Descriptors do not depend on whether a tile's triples are contracted by one
block or by two: ranges that take either way give the same bits."""
import numpy as np
import pytest

import mala_synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tj", [6, 8, 10])
def test_same_bits(tj):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_19617_amd as mala
    s = mala_synth.paper_solid()
    ctx = mala.Context(0)
    # 400 tiles: four rounds of half blocks, two of whole ones, so one block per tile
    whole = ctx.mala_descriptors(s.positions, s.L, s.N, s.rcut, tj, 0, 400 * 64)
    for tiles in (1, 64, 128, 300, 384):
        print("twojmax", tj, "tiles", tiles, flush=True)
        for short in (0, 1, 63):                        # points missing from the last tile
            n = tiles * 64 - short
            part = ctx.mala_descriptors(s.positions, s.L, s.N, s.rcut, tj, 0, n)
            assert torch.equal(part, whole[:n])
    ctx.check_device_errors()
    ctx.close()
