"""The fused execution of a plan's small steps, run on the host as the kernel
reads it: bounds, lifetimes, levels and the value against the plan run step by
step and, where small, brute force."""
import os
import subprocess

import pytest

import instances as I
from oracle import brute

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1805_00475_amd")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fuse") / "fuse_check")
    cmd = ["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "cpp", "fuse_check.cpp"), "-L", PKG, "-ltn", f"-Wl,-rpath,{PKG}", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _mixed(n, m, seed, max_len=9):
    f = I.random_mixed_formula(n, m, I.Rng(seed), max_len=max_len)
    return f


CASES = [
    ("1in3-n20", I.small_1in3(1)),
    ("one-clause", I.Formula(2, [(I.OR, [1, -2])])),
    ("unsat", I.Formula(3, [(I.OR, []), (I.OR, [1, 2, 3])])),
    ("free-variables", I.Formula(9, [(I.OR, [1, -2]), (I.EXACTLY_ONE, [4, 5, 4])])),
    ("cvc-n60", I.cvc(60, 0)),
    ("cvc-n90", I.cvc(90, 3)),
    ("1in3-n110", I.large_1in3(110, 0.62, 4)),
    # clauses of up to 9 literals and variables of many occurrences: initial
    # tensors of up to the fused rank and beyond
    ("mixed-long", _mixed(16, 9, 5)),
    ("wide-clause", I.Formula(16, [(I.OR, list(range(1, 17))), (I.XOR, [1, 5, -9])])),
    ("many-occurrences", I.Formula(20, [(I.OR, [1, k]) for k in range(2, 17)])),
    # disconnected components: a chain of scalars
    ("components", I.Formula(40, [(I.OR, [2 * k + 1, -(2 * k + 2)]) for k in range(20)])),
]


@pytest.mark.parametrize("name,f", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("es,wide", [(1, 0), (1, 1), (4, 0), (4, 1), (8, 0)])
def test_fused_execution(checker, tmp_path, name, f, es, wide):
    path = tmp_path / "f.txt"
    path.write_text(f"{f.n_vars} {len(f.clauses)}\n" +
                    "".join(f"{k} {len(c)} {' '.join(map(str, c))}\n" for k, c in f.clauses))
    for order in (0, 1):
        r = subprocess.run([checker, str(path), str(order), str(es), str(wide)], capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:]
        if f.n_vars <= 24:
            assert int(r.stdout.split("\n")[-3]) == brute.count(f)
