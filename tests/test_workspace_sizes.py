"""Workspace sizes of circuits with 2^8..2^10 copies: 2^9 copies take no scratch for
the matrix-core contraction (it uses tables that are free by then), so circuits up
to the static array of gkr_prove_circuit_noalloc keep fitting it. On the GPU such
circuits give the scalar contraction's proofs, with the scratch in those tables and
where they are too small for it."""
import numpy as np
import pytest

import gkr_synth as gs

gkr = pytest.importorskip("paper_2404_10404_amd.gkr")


def _spec(depth, copies, widths, seed=1):
    return gs.CircuitSpec(depth=depth, log_copies=copies, log_sub_width=widths, mu=(1, 2), seed=seed)


@pytest.mark.parametrize("depth,copies,widths,nbytes", [
    (10, 9, (10,) * 11, 236698880),
    (1, 9, (0, 12), 249058304),
    (4, 9, (9, 10, 2, 0, 10), 94167040),
    (3, 9, (8,) * 4, 32209408),
    (2, 10, (9, 9, 9), 140171264),  # scratch of its own
    (2, 8, (11, 11, 11), 102766336),
])
def test_workspace_bytes(depth, copies, widths, nbytes):
    spec = _spec(depth, copies, widths)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec))
    assert c.workspace_bytes == nbytes <= gkr.NOALLOC_WORKSPACE_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("depth,widths", [(10, (10,) * 11), (1, (0, 12)), (2, (7, 11, 8)), (2, (8, 9, 11))])
def test_static_workspace_proofs_equal_the_scalar_contraction(depth, widths):
    import torch
    spec = _spec(depth, 9, widths, seed=17)
    c = gkr.Circuit.from_synth(spec, gs.make_wiring(spec))
    inputs = gs.make_inputs(spec)
    d_in = gkr.device_elements(inputs)
    out = torch.zeros((1 << c.s(0), 8), dtype=torch.int32, device="cuda")
    proof = gkr.alloc_bytes(c.proof_bytes)
    print("no-alloc, 2^9 copies, widths %s" % (widths,), flush=True)
    n = gkr.prove_circuit_noalloc(c, d_in, spec.seed, out, proof)
    torch.cuda.synchronize()
    got = bytes(proof[:n].cpu().numpy().tobytes())
    p = gkr.Prover(c)
    p.ws.fill_(0xA5)
    try:
        gkr.set_contraction(False)
        p.prove(d_in, spec.seed)
        torch.cuda.synchronize()
    finally:
        gkr.set_contraction(True)
    assert got == p.proof_bytes()
    outs = np.ascontiguousarray(gkr.host_elements(out))
    assert np.array_equal(outs, gkr.host_elements(p.outputs))
    assert gkr.verify(c, inputs, outs, spec.seed, got) == 1
