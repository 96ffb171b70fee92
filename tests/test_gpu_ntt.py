"""Commitments whose transforms meet the edges of the NTT kernel: lengths on
either side of a tile (2^10 entries after the blow-up by four) and of a pass, with
the entries that bring the partly reduced butterflies to their bounds (0, 1 and
p - 1, alone or alternating), bit-exact against the oracle.
"""
import numpy as np
import pytest

from oracle import vpd

pytestmark = pytest.mark.gpu

P = 0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001


def _limbs(vals):
    return np.frombuffer(b"".join(int(v).to_bytes(32, "little") for v in vals), dtype=np.uint32).reshape(-1, 8).copy()


@pytest.mark.parametrize("log_n", [2, 7, 8, 9, 10])
@pytest.mark.parametrize("kind", ["top", "zero", "one-top", "top-last", "sparse"])
def test_commitment_of_bounding_vectors(log_n, kind):
    import torch
    from paper_2404_10404_amd import gkr
    n = 1 << log_n
    vals = {"top": [P - 1] * n, "zero": [0] * n, "one-top": [1 if k & 1 else P - 1 for k in range(n)],
            "top-last": [0] * (n - 1) + [P - 1], "sparse": [P - 1 if k % 5 == 0 else 0 for k in range(n)]}[kind]
    ws = gkr.alloc_bytes(gkr.vpd_workspace_bytes(log_n))
    root = gkr.alloc_bytes(32)
    gkr.vpd_commit(log_n, gkr.device_elements(_limbs(vals)), root, ws)
    torch.cuda.synchronize()
    assert bytes(root[:32].cpu().numpy().tobytes()) == vpd.commit(vals).root
