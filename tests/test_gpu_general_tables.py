"""General circuits on either side of the limits of the phase-2 table passes:
tables with the first round in their pass (above 2^14 entries) or without, and
source-block values with fewer columns than a workgroup has threads, as many, and
several column blocks. The host verifier accepts the proofs, and refuses them with
a bit of the last block value flipped.
"""
import numpy as np
import pytest

import gkr_synth as gs

pytestmark = pytest.mark.gpu

SHAPES = [
    # depth, n, sigmas, fan-in, reach
    (2, 0, (13, 13, 13), 2, 1),      # one column, phase 2 of 2^13 or 2^14 entries
    (2, 0, (14, 15, 14), 2, 2),
    (3, 3, (11, 12, 11, 12), 3, 3),  # eight columns, several blocks
    (2, 8, (6, 7, 6), 4, 2),         # as many columns as threads
    (3, 10, (5, 4, 5, 6), 4, 3),     # four column blocks
    (1, 15, (0, 0), 1, 1),           # columns only: the tables are one row
]


@pytest.mark.parametrize("shape", SHAPES)
def test_general_tables_verify(shape):
    import torch
    from paper_2404_10404_amd import gkr
    depth, n, sig, fanin, reach = shape
    spec = gs.GeneralSpec(depth=depth, log_copies=n, log_sub_width=sig, max_fanin=fanin, reach=reach, cross=(1, 2),
                          seed=301 + n)
    inputs = gs.make_general_inputs(spec)
    c = gkr.GeneralCircuit.from_synth(spec, gs.make_general_wiring(spec))
    pr = gkr.Prover(c)
    pr.prove(gkr.device_elements(inputs), spec.seed)
    torch.cuda.synchronize()
    proof = pr.proof_bytes()
    outs = np.ascontiguousarray(gkr.host_elements(pr.outputs))
    assert gkr.verify(c, inputs, outs, spec.seed, proof) == 1
    bad = bytearray(proof)
    bad[-32] ^= 1
    assert gkr.verify(c, inputs, outs, spec.seed, bytes(bad)) == 0
