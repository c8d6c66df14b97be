"""The plan check covers the fused layout as the kernel uses it: where programs
write their results, and their LDS places."""
import os
import subprocess

import pytest

import instances as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1805_00475_amd")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("verify") / "verify_check")
    cmd = ["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "cpp", "verify_check.cpp"), "-L", PKG, "-ltn", f"-Wl,-rpath,{PKG}", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


# one program, and several whose results larger steps read
@pytest.mark.parametrize("name,f", [("1in3-n20", I.small_1in3(1)), ("cvc-n60", I.cvc(60, 0)), ("cvc-n90", I.cvc(90, 3)),
                                    ("1in3-n110", I.large_1in3(110, 0.62, 4))])
@pytest.mark.parametrize("es", [1, 4, 8])
def test_verify_exec(program, tmp_path, name, f, es):
    path = tmp_path / "f.txt"
    path.write_text(f"{f.n_vars} {len(f.clauses)}\n" +
                    "".join(f"{k} {len(c)} {' '.join(map(str, c))}\n" for k, c in f.clauses))
    for order in (0, 1):
        r = subprocess.run([program, str(path), str(order), str(es)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:]
