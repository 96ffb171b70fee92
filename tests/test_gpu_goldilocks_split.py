"""Goldilocks phase 1 with the addition gates contracted over the copies against the
three-table form (gkr_set_contraction 0): proofs and outputs byte for byte, at the
edges of the rule (2^23 entries: fewest copies, fewest wires), with only ADD or only
MUL gates, and beside layers that keep the three tables. The switch takes effect:
the two forms make different launches."""
import ctypes

import numpy as np
import pytest

import gkr_synth as gs
from test_gpu_batch_forms import _Entry

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies,widths,mu", [
    (9, (14, 14), (1, 2)), (15, (8, 5, 8), (1, 4)), (10, (12, 13, 13), (1, 10)), (10, (11, 13), (0, 1)),
    (9, (13, 14), (1, 1)), (9, (7, 14, 9, 14), (3, 10)),
])
def test_equals_the_three_table_form(copies, widths, mu):
    import torch

    from paper_2404_10404_amd import gkr
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    spec = gs.CircuitSpec(depth=len(widths) - 1, log_copies=copies, log_sub_width=widths, mu=mu, seed=70 + copies)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec), gkr.FIELD_GOLDILOCKS)
    d_in = gkr.gl_device_elements(gs.make_goldilocks_inputs(spec))
    lib, got = gkr.lib(), []
    try:
        for contracted in (True, False):
            print("goldilocks copies 2^%d widths %s mu %s contracted %s" % (copies, widths, mu, contracted), flush=True)
            gkr.set_contraction(contracted)
            p = gkr.GlProver(c)
            p.ws.fill_(0xA5)
            torch.cuda.synchronize()
            assert lib.gkr_profile_enable(1) == 0
            p.prove(d_in, spec.seed)
            torch.cuda.synchronize()
            arr, n = (_Entry * 32)(), ctypes.c_uint32(0)
            assert lib.gkr_profile_read(arr, 32, ctypes.byref(n)) == 0
            lib.gkr_profile_enable(0)
            got.append((p.proof_bytes(), np.array(p.host_outputs()), sum(e.launches for e in arr[:n.value])))
            del p
    finally:
        gkr.set_contraction(True)
        lib.gkr_profile_enable(0)
    assert got[0][0] == got[1][0]
    assert np.array_equal(got[0][1], got[1][1])
    assert got[0][2] != got[1][2]
