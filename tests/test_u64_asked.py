"""64-bit arithmetic asked for is 64-bit arithmetic; only the automatic choice
runs wide 64-bit counts in small moduli."""
import pytest

from oracle import elim
from paper_1805_00475_amd import tn
from test_workspace_sizes import _wide


def test_workspace_is_a_64_bit_planes():
    _, net, plan = _wide()
    one = tn.workspace_bytes(net, plan, flags=tn.FLAG_NO_MFMA)
    for g in (0, 1, 16):
        assert tn.workspace_bytes(net, plan, arith="u64", prime_group=g) == one


@pytest.mark.gpu
def test_kernels():
    f, net, plan = _wide()
    want = elim.count_rns(f)
    for arith in ("u64", "auto"):
        print("[gpu case] arith", arith, flush=True)
        assert tn.count_plan(net, plan, arith=arith, flags=tn.FLAG_TIMING) == want
        # matrix-core launches are of residues, 64-bit planes come alone
        runs = [r for r in tn.launches() if r[0] in ("mfma", "narrow")]
        assert (runs == []) == (arith == "u64")
        assert (max(r[5] for r in tn.launches()) == 1) == (arith == "u64")
    assert tn.count_batch([f], "best", arith="u64", workspace_bytes_=8 << 30, flags=tn.FLAG_TIMING) == [want]
    assert all(r[0] not in ("mfma", "narrow") for r in tn.launches())
