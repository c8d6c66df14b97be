"""Steps over at most 32 shared entries: every width of the narrow side, all
orders of C's lowest bits, row walks longer than the grid."""
import numpy as np
import pytest

from paper_1805_00475_amd import tn

pytestmark = pytest.mark.gpu


def _deposit(x, mask):
    out, k = np.zeros_like(x), 0
    while mask:
        low = mask & -mask
        out |= np.where((x >> k) & 1, low, 0)
        mask ^= low
        k += 1
    return out


def _run(fA, fB, s, low, m, kind, seed, kernel="auto"):
    """low: the sides of C's lowest bits, from bit 0 on; the rest alternate."""
    rng = np.random.default_rng(seed)
    left, maskA = {"A": fA, "B": fB}, 0
    for b in range(fA + fB):
        side = low[b] if b < len(low) else "AB"[b % 2]
        if not left[side]:
            side = "B" if side == "A" else "A"
        left[side] -= 1
        maskA |= (side == "A") << b
    if kind == "max":  # the largest magnitude a centred residue takes
        A = np.full(1 << (fA + s), m // 2 if m > 255 else m // 2 + 1, np.uint32)
        B = np.full(1 << (fB + s), m // 2, np.uint32)
    else:
        A = rng.integers(0, m, size=1 << (fA + s)).astype(np.uint32)
        B = rng.integers(0, m, size=1 << (fB + s)).astype(np.uint32)
    print("[gpu case]", fA, fB, s, low, m, kind, flush=True)
    C = tn.step(A, fA + s, B, fB + s, s, maskA, prime=m, kernel=kernel)
    want = A.reshape(-1, 1 << s).astype(np.int64) @ B.reshape(-1, 1 << s).astype(np.int64).T % m
    cmask = (1 << (fA + fB)) - 1
    at = _deposit(np.arange(1 << fA), maskA)[:, None] | _deposit(np.arange(1 << fB), cmask ^ maskA)[None]
    assert np.array_equal(C[at], want)


@pytest.mark.parametrize("low", ["AA", "AB", "BA", "BB", "BBBBBB", "AAAAAAA"])
@pytest.mark.parametrize("s", range(6))
@pytest.mark.parametrize("fB", [4, 5, 6])
def test_few_rows_small_moduli(fB, s, low):
    _run(9, fB, s, low, 255, "uniform", 10 * fB + s)
    _run(11, fB, s, low, 251, "max", 1)


@pytest.mark.parametrize("m", [255, 65267])
@pytest.mark.parametrize("fA,fB,s", [(8, 0, 0), (8, 0, 1), (9, 1, 2), (10, 2, 3), (12, 3, 4), (8, 4, 5), (8, 3, 5),
                                     (21, 0, 1), (21, 1, 2), (16, 7, 0), (20, 3, 3)])
def test_streaming_walks(fA, fB, s, m):
    for low in ("AAAA", "BBBB", "AB"):
        _run(fA, fB, s, low, m, "max" if low == "AB" else "uniform", fA + fB)


@pytest.mark.parametrize("m", [255, 65267])
@pytest.mark.parametrize("s", [0, 1, 2, 3, 4, 5, 6, 7, 16, 17, 18])
def test_generic_row_lengths(s, m):
    # rows of less than one vector, of several, and of several exact ranges
    _run(3, 2, s, "AB", m, "uniform", s, "generic")
    _run(2, 1, s, "BA", m, "max", s, "generic")


@pytest.mark.parametrize("s", [0, 1, 2, 5, 17])
def test_generic_row_lengths_u64(s):
    rng = np.random.default_rng(s)
    A = rng.integers(0, 1 << 62, size=4 << s, dtype=np.uint64)
    B = rng.integers(0, 1 << 62, size=2 << s, dtype=np.uint64)
    C = tn.step(A, s + 2, B, s + 1, s, 0b011, kernel="generic")
    a, b = A.reshape(4, -1), B.reshape(2, -1)
    for xa in range(4):
        for xb in range(2):
            assert int(C[xa | xb << 2]) == sum(int(v) for v in a[xa] * b[xb]) % (1 << 64)
