"""Batches whose larger steps run as one chain of launches or as several side
by side (by the workspace): the same counts, also for more residue planes than
a launch takes."""
import json
import os

import pytest

import instances as I
from paper_1805_00475_amd import tn

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")


def _instances():
    out = []
    for name, n in (("cvc_counts.json", 120), ("cvc200_counts.json", 200)):
        items = [it for it in json.load(open(os.path.join(GOLD, name)))["items"] if it["n"] == n]
        out += [(I.cvc(n, it["seed"]), int(it["count"])) for it in items[:6 if n == 120 else 1]]
    gold = json.load(open(os.path.join(GOLD, "batch_counts.json")))["items"]
    return out + [(I.batch_instance(it["index"]), int(it["count"])) for it in gold[:20]]


# 4 GiB is the least workspace of four chains
@pytest.mark.parametrize("gib", [3, 4, 6])
@pytest.mark.parametrize("flags", [0, tn.FLAG_WIDE_RNS, tn.FLAG_TIMING, tn.FLAG_NO_MFMA])
def test_chains(gib, flags):
    many = _instances()
    print("[gpu case] batch chains", gib, "GiB flags", flags, flush=True)
    got = tn.count_batch([f for f, _ in many], "best", flags=flags, workspace_bytes_=gib << 30,
                         workspace=tn.Workspace())
    assert got == [c for _, c in many]
