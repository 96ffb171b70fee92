"""Statements whose two vectors take different numbers of digest levels, on either
side of the level size from which a chunk goes to a thread (512 chunks of 1 KiB):
the host verifier, which digests both vectors by itself, accepts the proofs, and
refuses one for an output vector with a bit flipped in its last element.
"""
import numpy as np
import pytest

import gkr_synth as gs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sig_out,sig_in", [(1, 14), (14, 15), (15, 4), (16, 15), (15, 10)])
@pytest.mark.parametrize("field", ["bn254", "goldilocks"])
def test_statement_digests(field, sig_out, sig_in):
    import torch
    from paper_2404_10404_amd import gkr
    extra = 2 if field == "goldilocks" else 0  # elements a quarter as long
    spec = gs.CircuitSpec(depth=1, log_copies=extra, log_sub_width=(sig_out, sig_in), mu=(1, 2), seed=500 + sig_in)
    wiring = gs.make_wiring(spec)
    if field == "bn254":
        c, inputs = gkr.Circuit.from_synth(spec, wiring), gs.make_inputs(spec)
        p = gkr.Prover(c)
        p.prove(gkr.device_elements(inputs), spec.seed)
        torch.cuda.synchronize()
        outs, verify = np.ascontiguousarray(gkr.host_elements(p.outputs)), gkr.verify
    else:
        c, inputs = gkr.Circuit.from_synth(spec, wiring, gkr.FIELD_GOLDILOCKS), gs.make_goldilocks_inputs(spec)
        p = gkr.GlProver(c)
        p.prove(gkr.gl_device_elements(inputs), spec.seed)
        torch.cuda.synchronize()
        outs, verify = np.ascontiguousarray(p.host_outputs()), gkr.gl_verify
    proof = p.proof_bytes()
    assert verify(c, inputs, outs, spec.seed, proof) == 1
    bad = outs.copy()
    bad.reshape(-1)[-1 if field == "goldilocks" else -8] ^= 1
    assert verify(c, inputs, bad, spec.seed, proof) == 0
