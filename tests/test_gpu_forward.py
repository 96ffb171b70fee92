"""Outputs of one-layer circuits whose input table is above the size from which the
forward pass goes in column blocks, or just below: sampled outputs (both ends of
the rows and the edges of the 2^8-column blocks) against integer arithmetic.
"""
import numpy as np
import pytest

import gkr_synth as gs

pytestmark = pytest.mark.gpu

P = 0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001


@pytest.mark.parametrize("n,sig_out,sig_in", [(9, 13, 13), (9, 12, 14), (10, 14, 13), (12, 9, 11), (8, 13, 15)])
def test_forward_outputs(n, sig_out, sig_in):
    import torch
    from paper_2404_10404_amd import gkr
    spec = gs.CircuitSpec(depth=1, log_copies=n, log_sub_width=(sig_out, sig_in), mu=(1, 2), seed=400 + n)
    wiring = gs.make_wiring(spec)
    inputs = np.ascontiguousarray(gs.make_inputs(spec))
    pr = gkr.Prover(gkr.Circuit.from_synth(spec, wiring))
    pr.prove(gkr.device_elements(inputs), spec.seed)
    torch.cuda.synchronize()
    outs = np.ascontiguousarray(gkr.host_elements(pr.outputs))
    as_int = lambda a, i: int.from_bytes(a[i].tobytes(), "little")
    ncop = 1 << n
    rng = np.random.default_rng(n)
    cols = sorted({0, 1, 63, 64, 127, 128, 255, ncop - 1} | {256 % ncop, 257 % ncop, (ncop >> 1) - 1})
    rows = [0, 1, (1 << sig_out) - 1] + [int(z) for z in rng.integers(0, 1 << sig_out, 40)]
    types, xs, ys = wiring[0].kind, wiring[0].x, wiring[0].y
    for z in rows:
        for c in cols:
            a, b = as_int(inputs, int(xs[z]) * ncop + c), as_int(inputs, int(ys[z]) * ncop + c)
            want = (a * b if int(types[z]) == gs.GATE_MUL else a + b) % P
            assert as_int(outs, z * ncop + c) == want, (z, c)
