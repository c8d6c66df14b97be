"""A plan carries the fused execution of its default arithmetic, also where
the search lowered its count bound (from 16-bit primes to small moduli)."""
import os
import subprocess

import pytest

import instances as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1805_00475_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("exec") / "exec_check")
    cmd = ["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "cpp", "exec_check.cpp"), "-L", PKG, "-ltn", f"-Wl,-rpath,{PKG}", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _long(free):
    """Nine 3-CNF formulas of 40 variables side by side and ``free`` variables:
    a bound two bits above the tightened one."""
    clauses = []
    for i in range(9):
        clauses += [(I.OR, [v + 40 * i for v in c]) for _, c in I.exactly_one_3(40, 60, I.Rng(i)).clauses]
    return I.Formula(360 + free, clauses)


@pytest.mark.parametrize("name,f,lowered", [
    ("long-28", _long(28), True),
    ("long-29", _long(29), True),
    ("cvc-n60", I.cvc(60, 0), False),
    ("cvc-n90", I.cvc(90, 1), False),
    ("1in3-n20", I.small_1in3(1), False),
])
def test_default_execution_is_kept(program, tmp_path, name, f, lowered):
    path = tmp_path / "f.txt"
    path.write_text(f"{f.n_vars} {len(f.clauses)}\n" +
                    "".join(f"{k} {len(c)} {' '.join(map(str, c))}\n" for k, c in f.clauses))
    # (4: the search of many orders, on two threads, one round)
    r = subprocess.run([program, str(path), "4", "2", "1"], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout
    assert ("lowered" in r.stdout) == lowered, r.stdout
