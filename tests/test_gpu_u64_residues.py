"""64-bit counts of plans with wide steps run in small moduli: the same counts
as the 64-bit kernels, from the smallest such plan up, in the workspace a
64-bit plane needs, and in batches."""
import ctypes

import pytest

import instances as I
from oracle import elim
from paper_1805_00475_amd import tn

pytestmark = pytest.mark.gpu
ROUTE_MACS = 2 ** 25


def _cnf3(n, m, seed):
    rng = I.Rng(seed)
    f = I.exactly_one_3(n, m, rng)
    f.clauses = [(I.OR, [v if rng.coin() else -v for v in c]) for _, c in f.clauses]
    return f


def _count_in(net, plan, nbytes, flags=0, **kw):
    """tn_count with a workspace of exactly nbytes."""
    import torch
    buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    o = tn._opts(kw.get("arith", "auto"), 0, buf.data_ptr(), nbytes, tn.current_stream_handle(),
                 kw.get("prime_group", 0), flags)
    limbs, n = (ctypes.c_uint32 * 80)(), ctypes.c_size_t()
    st = tn.load().tn_count(net.h, plan.h, ctypes.byref(o), limbs, 80, ctypes.byref(n))
    return st, tn._limbs_to_int(limbs, n.value) if st == 0 else None


# below and above the route's least multiply-adds, up to rank 22
@pytest.mark.parametrize("n,m,seed", [(36, 40, 1), (40, 46, 3), (40, 48, 2), (50, 60, 1)])
def test_counts_agree(n, m, seed):
    f = _cnf3(n, m, seed)
    net = tn.Network(f)
    plan = net.order("best", seed, rounds=1)
    print("[gpu case] 3-CNF", n, m, "macs %.2e" % plan.stats["macs"], flush=True)
    want = elim.count_rns(f)
    assert tn.count_plan(net, plan) == want
    assert tn.count_plan(net, plan, arith="u64", prime_group=1) == want
    assert tn.count_plan(net, plan, flags=tn.FLAG_NO_MFMA) == want
    # the results keep their type: one 64-bit value, no moduli
    assert tn.contract(net, plan) == want and tn.moduli(plan) == []


def test_tight_workspace():
    # what one 64-bit plane takes (the moduli in groups), and a byte less
    # than any layout takes
    f = _cnf3(50, 60, 1)
    net = tn.Network(f)
    plan = net.order("best", 1, rounds=1)
    assert plan.stats["macs"] >= ROUTE_MACS
    want = tn.count_plan(net, plan)
    one = tn.workspace_bytes(net, plan, flags=tn.FLAG_NO_MFMA)
    print("[gpu case] tight workspace", one, flush=True)
    assert _count_in(net, plan, one) == (0, want)
    assert _count_in(net, plan, one, prime_group=1) == (0, want)
    assert _count_in(net, plan, 4 << 20)[0] == -4


def test_batch_agrees():
    fs = [_cnf3(40, 46, 3), I.small_1in3(4), _cnf3(40, 48, 2), I.cvc(60, 1)]
    want = [tn.count(f, "best", flags=tn.FLAG_NO_MFMA) for f in fs]
    assert tn.count_batch(fs, "best", workspace_bytes_=4 << 30) == want
