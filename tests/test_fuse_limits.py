"""Long sparse formulas: a program's tensors and its text (steps, items,
levels) together stay within a work-group's LDS, for every entry size."""
import os
import subprocess

import pytest

import instances as I

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1805_00475_amd")
LDS = 160 << 10  # bytes a work-group may ask for on gfx950


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("fuse") / "fuse_check")
    cmd = ["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(ROOT, "tests", "cpp", "fuse_check.cpp"), "-L", PKG, "-ltn", f"-Wl,-rpath,{PKG}", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _units(n):
    return I.Formula(n, [(I.OR, [v if v % 3 else -v]) for v in range(1, n + 1)])


def _path(n, kind, block):
    """Chains of 2-literal clauses over blocks of ``block`` variables."""
    return I.Formula(n, [(kind, [v, v + 1]) for v in range(1, n) if v % block])


CASES = [
    ("units-2000", _units(2000)),
    ("units-3000", _units(3000)),
    ("parity-path-2400", _path(2400, I.XOR, 10 ** 9)),
    ("parity-path-3000", _path(3000, I.XOR, 10 ** 9)),
    ("parity-chains-70x36", _path(70 * 36, I.XOR, 36)),
    ("or-chains-20x120", _path(2400, I.OR, 120)),
]


@pytest.mark.parametrize("name,f", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("es", [1, 4, 8])
def test_program_fits_lds(program, tmp_path, name, f, es):
    path = tmp_path / "f.txt"
    path.write_text(f"{f.n_vars} {len(f.clauses)}\n" +
                    "".join(f"{k} {len(c)} {' '.join(map(str, c))}\n" for k, c in f.clauses))
    for order in (0, 1):
        r = subprocess.run([program, str(path), str(order), str(es), "0"], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:]
        assert int(r.stdout.split(" lds ")[1].split(",")[0]) <= LDS, r.stdout


def _chains(blocks):
    """Disjoint chains of 36 variables of unlike neighbours, two solutions
    each, and one chain of 40 in clauses of two literals, F(42) solutions."""
    f = _path(36 * blocks + 40, I.XOR, 36)
    f.clauses = [c for c in f.clauses if c[1][0] <= 36 * blocks]
    f.clauses += [(I.OR, [36 * blocks + k, 36 * blocks + k + 1]) for k in range(1, 40)]
    return f, 2 ** blocks * 267914296


def test_chains_take_more_than_64_kib(program, tmp_path):
    # the formula of the GPU test below
    for es in (1, 4):
        f, _ = _chains(60)
        path = tmp_path / "f.txt"
        path.write_text(f"{f.n_vars} {len(f.clauses)}\n" +
                        "".join(f"{k} {len(c)} {' '.join(map(str, c))}\n" for k, c in f.clauses))
        r = subprocess.run([program, str(path), "0", str(es), "0"], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:]
        assert 64 << 10 < int(r.stdout.split(" lds ")[1].split(",")[0]) <= LDS, r.stdout


@pytest.mark.gpu
def test_long_formulas_on_the_gpu():
    from paper_1805_00475_amd import tn
    f, want = _chains(60)
    net = tn.Network(f)
    plan = net.order("greedy", 0)
    for flags in (0, tn.FLAG_WIDE_RNS):
        mods = tn.moduli(plan, flags=flags)
        print("[gpu case] chains, planes", len(mods), flush=True)
        assert (max(mods) > 255) == (flags != 0)
        assert tn.count_plan(net, plan, flags=flags) == want
    # 64-bit counts: 600 constant weights beside a path of 40 variables
    c = I.CSP(40, [2] * 40, [((), [1])] * 600 + [((v, v + 1), [0, 1, 1, 1]) for v in range(1, 40)])
    net = tn.Network(c)
    plan = net.order("greedy", 0)
    print("[gpu case] 64-bit counts of", 679, "tensors", flush=True)
    assert tn.moduli(plan) == [] and tn.count_plan(net, plan) == 267914296
    many = [(f, want), (I.cvc(60, 0), tn.count(I.cvc(60, 0))), (_units(3000), 1)]
    print("[gpu case] batch with long formulas", flush=True)
    assert tn.count_batch([m for m, _ in many], "greedy", workspace_bytes_=8 << 30) == [w for _, w in many]
