"""The wave-wide hashing routines (csrc/sha256_wave.hpp) against hashlib and the
oracle's compression function: whole digests, every bit. The words include
all zeros, all ones and single bits, so every carry of the split schedule and
of the two lane groups is met."""
import ctypes
import hashlib
import os
import random

import numpy as np
import pytest

from oracle import transcript as ot

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "libwavecheck.so")


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    if not os.path.exists(LIB):
        raise ImportError("tests/native/libwavecheck.so is not built; run __graft_entry__.build()")
    L = ctypes.CDLL(LIB)
    vp, u32 = ctypes.c_void_p, ctypes.c_uint32
    L.wavecheck_sha_chain.argtypes = [vp, vp, vp, u32, u32, ctypes.c_int]
    L.wavecheck_sha_message.argtypes = [vp, vp, u32, ctypes.c_int]
    return L


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.uint32).view(np.int32)).cuda()


def _words(rng, count):
    special = [0, 0xFFFFFFFF, 0x80000000, 1, 0x55555555]
    return [rng.choice(special) if rng.random() < 0.3 else rng.getrandbits(32) for _ in range(count)]


@pytest.mark.parametrize("length", [9, 11, 17])
def test_message_digests(lib, length):
    import torch
    rng = random.Random(length)
    msgs = [[0] * length, [0xFFFFFFFF] * length] + [_words(rng, length) for _ in range(30)]
    out = torch.zeros(8 * len(msgs), dtype=torch.int32, device="cuda")
    assert lib.wavecheck_sha_message(_dev(msgs).data_ptr(), out.data_ptr(), len(msgs), length) == 0
    got = out.cpu().numpy().view(np.uint32).reshape(-1, 8)
    for m, g in zip(msgs, got):
        want = hashlib.sha256(b"".join(w.to_bytes(4, "big") for w in m)).digest()
        assert b"".join(int(x).to_bytes(4, "big") for x in g) == want


@pytest.mark.parametrize("helped", [0, 1])
def test_chained_compressions(lib, helped):
    import torch
    rng = random.Random(7 + helped)
    cases, rounds = 40, 5
    st = [_words(rng, 8) for _ in range(cases)]
    blocks = [[_words(rng, 16) for _ in range(rounds)] for _ in range(cases)]
    out = torch.zeros(8 * cases, dtype=torch.int32, device="cuda")
    assert lib.wavecheck_sha_chain(_dev(st).data_ptr(), _dev(blocks).data_ptr(), out.data_ptr(), cases, rounds,
                                   helped) == 0
    got = out.cpu().numpy().view(np.uint32).reshape(-1, 8)
    for s, bl, g in zip(st, blocks, got):
        state = b"".join(w.to_bytes(4, "big") for w in s)
        for b in bl:
            state = ot.compress(state, b"".join(w.to_bytes(4, "big") for w in b))
        assert b"".join(int(x).to_bytes(4, "big") for x in g) == state
