"""What tn_workspace_bytes answers for 64-bit counts that run in small moduli:
one 64-bit plane unless several planes are asked for, and the same count in any
workspace that the call takes."""
import ctypes

import pytest

import instances as I
from oracle import elim
from paper_1805_00475_amd import tn


def _wide(n=40, m=48, seed=2):
    rng = I.Rng(seed)
    f = I.exactly_one_3(n, m, rng)
    f.clauses = [(I.OR, [v if rng.coin() else -v for v in c]) for _, c in f.clauses]
    net = tn.Network(f)
    plan = net.order("best", seed, rounds=1)
    assert plan.stats["macs"] >= 2 ** 25 and tn.moduli(plan) == []
    return f, net, plan


def test_one_plane_unless_asked():
    _, net, plan = _wide()
    one = tn.workspace_bytes(net, plan, flags=tn.FLAG_NO_MFMA)   # the 64-bit plane
    assert tn.workspace_bytes(net, plan) == one
    assert tn.workspace_bytes(net, plan, prime_group=1) == one
    # k residue planes, as the same counts asked for as residues
    k = len(tn.moduli(plan, arith="rns"))
    assert k > 2
    for g in range(2, k + 2):
        rns = tn.workspace_bytes(net, plan, arith="rns", prime_group=g)
        assert one <= tn.workspace_bytes(net, plan, prime_group=g) <= max(one, rns)


@pytest.mark.gpu
@pytest.mark.parametrize("n,m,seed", [(40, 48, 2), (44, 52, 3), (50, 60, 1)])
def test_counts_in_any_workspace(n, m, seed):
    import torch
    f, net, plan = _wide(n, m, seed)
    want = elim.count_rns(f)
    k = len(tn.moduli(plan, arith="rns"))
    sizes = {tn.workspace_bytes(net, plan), tn.workspace_bytes(net, plan, flags=tn.FLAG_NO_MFMA)}
    sizes |= {tn.workspace_bytes(net, plan, arith="rns", prime_group=g) for g in range(1, k + 1)}
    for nbytes in sorted(sizes):
        print("[gpu case] 3-CNF", n, m, "workspace", nbytes, flush=True)
        buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        o = tn._opts("auto", 0, buf.data_ptr(), nbytes, tn.current_stream_handle(), 0, 0)
        limbs, nl = (ctypes.c_uint32 * 80)(), ctypes.c_size_t()
        assert tn.load().tn_count(net.h, plan.h, ctypes.byref(o), limbs, 80, ctypes.byref(nl)) == 0
        assert tn._limbs_to_int(limbs, nl.value) == want
    # (instances that do not share the workspace run alone)
    assert tn.count_batch([f, f], "best", workspace_bytes_=48 << 20, workspace=tn.Workspace()) == [want, want]
