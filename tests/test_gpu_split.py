"""Phase 1 with the addition gates contracted over the copies (csrc/gkr_split.hip,
wide layers of many copies) against the three-table form of the same library,
which the parity tests hold to the oracle: proofs and outputs byte for byte,
and the library's verifier accepts. Shapes at the edges of the rule (2^23
entries: fewest copies, fewest wires, as many MUL gates as it takes), layers of
other widths beside such a layer (so both forms meet in one proof), and only MUL
or only ADD gates (no addition term, or a MUL table without a nonzero row)."""
import numpy as np
import pytest

import gkr_synth as gs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies,widths,mu", [
    (9, (14, 14), (49, 100)), (13, (10, 10, 10), (3, 10)), (10, (12, 13, 13), (1, 10)), (9, (13, 14), (1, 1)),
    (10, (11, 13), (0, 1)), (9, (7, 14, 9, 14), (1, 4)), (9, (15, 15), (7, 10)),
])
def test_equals_the_three_table_form(copies, widths, mu):
    import torch

    from paper_2404_10404_amd import gkr
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    spec = gs.CircuitSpec(depth=len(widths) - 1, log_copies=copies, log_sub_width=widths, mu=mu, seed=90 + copies)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec))
    inputs = gs.make_inputs(spec)
    d_in = gkr.device_elements(inputs)
    got = []
    try:
        for contracted in (True, False):
            print("copies 2^%d widths %s mu %s contracted %s" % (copies, widths, mu, contracted), flush=True)
            gkr.set_contraction(contracted)
            p = gkr.Prover(c)
            p.ws.fill_(0xA5)  # nothing may be read before it is written
            p.prove(d_in, spec.seed)
            torch.cuda.synchronize()
            got.append((p.proof_bytes(), np.ascontiguousarray(gkr.host_elements(p.outputs))))
            del p
    finally:
        gkr.set_contraction(True)
    assert got[0][0] == got[1][0]
    assert np.array_equal(got[0][1], got[1][1])
    assert gkr.verify(c, inputs, got[0][1], spec.seed, got[0][0]) == 1


@pytest.mark.parametrize("copies,widths,mu", [
    (9, (14, 14), (1, 2)), (13, (10, 10), (3, 10)), (10, (12, 13), (0, 1)), (9, (13, 14), (1, 1)),
    (15, (8, 5, 8), (1, 4)),
])
def test_goldilocks_proofs_are_accepted(copies, widths, mu):
    """The same form over the Goldilocks field: the verifier, which evaluates the
    wiring predicates and the inputs itself, accepts (a wrong round sum is
    rejected but for a chance below 2^-50). 2^23 entries and more."""
    import torch

    from paper_2404_10404_amd import gkr
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    spec = gs.CircuitSpec(depth=len(widths) - 1, log_copies=copies, log_sub_width=widths, mu=mu, seed=50 + copies)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec), gkr.FIELD_GOLDILOCKS)
    inputs = gs.make_goldilocks_inputs(spec)
    p = gkr.GlProver(c)
    p.ws.fill_(0xA5)
    print("goldilocks copies 2^%d widths %s mu %s" % (copies, widths, mu), flush=True)
    p.prove(gkr.gl_device_elements(inputs), spec.seed)
    torch.cuda.synchronize()
    proof = p.proof_bytes()
    assert gkr.gl_verify(c, inputs, p.host_outputs(), spec.seed, proof) == 1
    bad = bytearray(proof)
    bad[8] ^= 1
    assert gkr.gl_verify(c, inputs, p.host_outputs(), spec.seed, bytes(bad)) == 0
