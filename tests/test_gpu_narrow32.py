"""Steps with at most 64 B rows modulo 16-bit primes against the oracle's sums."""
import numpy as np
import pytest

from paper_1805_00475_amd import tn
from test_gpu_kernels import P, _check

pytestmark = pytest.mark.gpu

# (rA, rB, s): every B block count (fB 0, 3, 4, 5, 6), A sides of less than one
# row tile, K from one chunk to many ranges, single outputs and the split-K dot's
# neighbours, and A and B exchanged
SHAPES = [(6, 6, 6), (12, 6, 6), (9, 9, 6), (14, 9, 6), (15, 10, 6), (16, 12, 7), (13, 12, 7), (14, 13, 8),
          (12, 12, 6), (13, 13, 7), (17, 10, 6), (20, 15, 11), (13, 12, 10), (13, 13, 10), (18, 17, 15),
          (11, 12, 9), (10, 16, 8), (21, 22, 16), (12, 11, 10), (9, 9, 9)]


@pytest.mark.parametrize("rA,rB,s", SHAPES)
def test_narrow32(rA, rB, s):
    for i, kind in enumerate(("uniform", "max", "half")):
        _check(rA, rB, s, "auto", P[i * 3], seed=rA * 31 + rB * 5 + s + i, kind=kind, samples=1500)


def test_narrow32_exact_range():
    # 2^19 outputs leave no scratch for K ranges, so the sums over K = 2^16 are
    # reduced once in the middle: largest negative residues against mixed ones
    p, s = P[0], 16
    rng = np.random.default_rng(3)
    A = np.full(1 << 30, p // 2 + 1, np.uint32)
    A[-(1 << s):] = rng.integers(0, p, size=1 << s, dtype=np.uint32)
    B = np.full(1 << 21, p // 2 + 1, np.uint32)
    B[1 << s:2 << s] = rng.integers(0, p, size=1 << s, dtype=np.uint32)
    maskA = ((1 << 14) - 1) << 5
    C = tn.step(A, 30, B, 21, s, maskA, prime=p).reshape(1 << 14, 32)
    b = B.reshape(32, 1 << s).astype(object)
    for xa in (0, 1, 63, 8191, (1 << 14) - 1):
        a = A[xa << s:(xa + 1) << s].astype(object)
        for j in (0, 1, 31):
            assert int(C[xa, j]) == int((a * b[j]).sum() % p)
