"""Goldilocks proofs of layers with many wires and few copies, where the local
values take one workgroup or several and a wave of the copy contraction has a
product per lane or fewer: the verifier, which evaluates the wiring predicates and
the inputs itself, accepts, and a changed proof is rejected."""
import pytest

import gkr_synth as gs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies,widths", [
    (0, (14, 14)), (0, (15, 15, 14)), (1, (14, 16)), (0, (17, 17)), (3, (14, 15)), (6, (12, 13)), (7, (12, 13)),
    (0, (18, 21)),
])
def test_tall_layers(copies, widths):
    import torch

    from paper_2404_10404_amd import gkr
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    spec = gs.CircuitSpec(depth=len(widths) - 1, log_copies=copies, log_sub_width=widths, mu=(1, 2), seed=60 + copies)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec), gkr.FIELD_GOLDILOCKS)
    inputs = gs.make_goldilocks_inputs(spec)
    p = gkr.GlProver(c)
    p.ws.fill_(0xA5)
    print("goldilocks copies 2^%d widths %s" % (copies, widths), flush=True)
    for _ in range(2):  # the counters are back at zero
        p.proof.zero_()
        p.prove(gkr.gl_device_elements(inputs), spec.seed)
        torch.cuda.synchronize()
        proof = p.proof_bytes()
        assert gkr.gl_verify(c, inputs, p.host_outputs(), spec.seed, proof) == 1
    bad = bytearray(proof)
    bad[8] ^= 1
    assert gkr.gl_verify(c, inputs, p.host_outputs(), spec.seed, bytes(bad)) == 0
