"""Steps over 128 to 512 shared entries that keep one side's rows in registers,
against exact products in double precision: every order of C's two lowest bits
(either side resident, words paired or not), the fewest rows on either side,
runs of one and of several tiles."""
import numpy as np
import pytest

from paper_1805_00475_amd import tn
from test_gpu_short_steps import _deposit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("low", ["AA", "AB", "BA", "BB"])
@pytest.mark.parametrize("fA,fB,s", [(17, 8, 7), (13, 12, 7), (9, 16, 7), (17, 8, 8), (13, 12, 8), (9, 16, 8),
                                     (19, 9, 9)])
def test_resident_rows(fA, fB, s, low):
    rng = np.random.default_rng(fA * 100 + s)
    m = 255 if low != "BA" else 254
    sides = list(low) + list(rng.permutation(["A"] * (fA - low.count("A")) + ["B"] * (fB - low.count("B"))))
    maskA = sum(1 << b for b, side in enumerate(sides) if side == "A")
    A = rng.integers(0, m, size=(1 << fA, 1 << s), dtype=np.uint32)
    B = rng.integers(0, m, size=(1 << fB, 1 << s), dtype=np.uint32)
    A[:70] = m // 2        # the largest sums a centred residue's products take
    B[-70:] = m // 2
    A[-300:] = m // 2 + 1
    print("[gpu case]", fA, fB, s, low, m, flush=True)
    C = tn.step(A.reshape(-1), fA + s, B.reshape(-1), fB + s, s, maskA, prime=m)
    dA = _deposit(np.arange(1 << fA), maskA)
    dB = _deposit(np.arange(1 << fB), ((1 << (fA + fB)) - 1) ^ maskA)
    Bt = B.astype(np.float64).T
    blocks = range(0, 1 << fA, 1 << 12)
    for r0 in blocks if s < 9 else (0, 13 << 12, 64 << 12, (1 << fA) - (1 << 12)):
        rows = slice(r0, r0 + (1 << 12))
        want = np.fmod(A[rows].astype(np.float64) @ Bt, m)
        assert np.array_equal(C[dA[rows, None] | dB[None]], want)
