"""The integer arithmetic that ends a matrix-core contraction, on the host against
Python integers: band sums at their bound (every byte of every term 255) for 2^0 to
2^24 terms, constant columns at the counts where a band shifted by three bytes
passes 64 bits, and random ones."""
import os
import random
import subprocess

import pytest

P = 0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001
RINV = pow(1 << 256, -1, P)
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("cc") / "cc_sum_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "native", "cc_sum_check.cpp")],
                   check=True)
    return exe


def _pairs(k):
    return min(k, 62 - k) + 1


@pytest.mark.parametrize("log_terms", [0, 12, 14, 19, 20, 21, 22, 24])
def test_band_sums_up_to_their_bound(checker, log_terms):
    rng = random.Random(log_terms)
    n = 1 << log_terms
    rows = [[_pairs(k) * 255 * 255 * n for k in range(63)]]
    # every term the same two elements, as in a column of equal copies
    for _ in range(8):
        u, w = (rng.randrange(P).to_bytes(32, "little") for _ in range(2))
        rows.append([n * sum(u[i] * w[k - i] for i in range(32) if 0 <= k - i < 32) for k in range(63)])
    rows += [[rng.randrange(_pairs(k) * 255 * 255 * n + 1) for k in range(63)] for _ in range(8)]
    top = pow(2, 508, P)
    lines = [" ".join(str(top >> (32 * i) & 0xFFFFFFFF) for i in range(8))]
    lines += [" ".join(map(str, r)) for r in rows]
    out = subprocess.run([checker], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
    assert [int(x, 16) for x in out.split()] == [sum(e << (8 * k) for k, e in enumerate(r)) * RINV % P for r in rows]


def test_power_of_two_that_folds_the_top_bits(checker):
    out = subprocess.run([checker, "constant"], capture_output=True, text=True, check=True).stdout
    assert sum(int(x) << (32 * i) for i, x in enumerate(out.split())) == pow(2, 508, P)
