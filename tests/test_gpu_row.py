"""The quadratic with a limb per lane (csrc/fr_row.hpp) against integer arithmetic:
random values, the ends of the range, and limbs of all ones and all zeros, which
run a carry or a borrow through every lane of a row."""
import ctypes
import os
import random

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = 0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001
LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libwavecheck.so")


def _cases(kind):
    rng = random.Random(len(kind))
    edge = [0, 1, P - 1, P - 2, (1 << 253) - 1, (1 << 224) - 1, 1 << 224, (1 << 32) - 1, P >> 1, (P >> 32) << 32]
    pick = (lambda: rng.choice(edge)) if kind == "edges" else (lambda: rng.randrange(P))
    if kind == "same":
        return [[e] * 4 for e in edge] + [[e, 0, e, 0] for e in edge[:6]]
    return [[pick() for _ in range(4)] for _ in range(256)]


@pytest.mark.parametrize("kind", ["random", "edges", "same"])
def test_row_quadratic(kind):
    import torch
    if not os.path.exists(LIB):
        raise ImportError("tests/native/libwavecheck.so is not built; run __graft_entry__.build()")
    lib = ctypes.CDLL(LIB)
    lib.wavecheck_row_quadratic.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_uint32]
    cases = _cases(kind)
    assert len(cases) % 4 == 0
    raw = np.frombuffer(b"".join(v.to_bytes(32, "little") for c in cases for v in c), dtype=np.int32).copy()
    d_in = torch.from_numpy(raw).cuda()
    out = torch.zeros(8 * len(cases), dtype=torch.int32, device="cuda")
    assert lib.wavecheck_row_quadratic(d_in.data_ptr(), out.data_ptr(), len(cases) // 4) == 0
    got = out.cpu().numpy().reshape(-1, 8)
    rinv = pow(1 << 256, -1, P)
    for (r, v0, v1, c2), g in zip(cases, got):
        want = (v0 + r * rinv * (v1 - v0 - c2 + r * rinv * c2)) % P
        assert int.from_bytes(g.tobytes(), "little") == want, (hex(r), hex(v0), hex(v1), hex(c2))
