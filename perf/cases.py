"""Measured cases of the counter: what its users have it do, over the sizes
of this repository's own workloads.

Three kinds of work, each through the public entry points of
``paper_1805_00475_amd.tn``:

* ``count``: the exact count of one formula or weighted network. The network
  and its contraction order are in hand (a program keeps both) except where
  ``whole`` is set, where one call builds, orders, contracts and recombines.
* ``batch``: ``count_batch`` of many formulas of uneven size, whole path.
* ``scorer``: the perceptron that scores contraction pairs: a training step
  (forward, listwise-loss backward, Adam) or the forward pass alone.

A case fixes the graph of a formula (``index``), the seed fixes its data:
literal signs, clause weights, batch members, features and labels. So every
seed contracts the same shapes with other values.
"""
import math
import random

import numpy as np
import torch

import instances as I
from paper_1805_00475_amd import tn
from paper_1805_00475_amd.train_order import init_params

LIMBS = 64           # 32-bit limbs a count is returned in (at most 2^2000)
MAX_PREDICTED_US = 1.5e5    # largest predicted device time of a drawn count
MAX_WORKSPACE = 80 << 30    # and its largest workspace
FEATURES, HIDDEN = 10, 128
ROWS_PER_GROUP = 208  # candidate pairs per state in the shipped training set


def listed():
    return [
        # one small formula counted in one call: 1-in-3 with 20 variables and
        # 14 clauses, the smallest workload (64-bit counts, call latency)
        {"name": "1in3-n20-call", "kind": "count", "family": "1in3", "n": 20, "m": 14, "index": 1, "order": "greedy",
         "rounds": 0, "arith": "auto", "whole": True},
        # a small vertex cover count (64-bit counts, 149 small steps)
        {"name": "cvc-n60", "kind": "count", "family": "cvc", "n": 60, "m": 0, "index": 0, "order": "greedy",
         "rounds": 0, "arith": "auto", "whole": False},
        # 3-CNF with 60 variables: 64-bit counts over a wide intermediate
        {"name": "3cnf-n60", "kind": "count", "family": "3cnf", "n": 60, "m": 72, "index": 1, "order": "best",
         "rounds": 1, "arith": "auto", "whole": False},
        # vertex cover at 120 variables: small moduli, mostly small steps
        {"name": "cvc-n120", "kind": "count", "family": "cvc", "n": 120, "m": 0, "index": 0, "order": "best",
         "rounds": 1, "arith": "auto", "whole": False},
        # vertex cover at the paper's largest size
        {"name": "cvc-n200", "kind": "count", "family": "cvc", "n": 200, "m": 0, "index": 1, "order": "best",
         "rounds": 1, "arith": "auto", "whole": False},
        # the same size in 16-bit primes (what counts past 332 bits use)
        {"name": "cvc-n200-primes", "kind": "count", "family": "cvc", "n": 200, "m": 0, "index": 0, "order": "best",
         "rounds": 1, "arith": "primes", "whole": False},
        # weighted independent sets of a cubic graph with 100 vertices:
        # weights reduced per prime, a count of about 1000 bits
        {"name": "hardcore-n100", "kind": "count", "family": "hardcore", "n": 100, "m": 0, "index": 5,
         "order": "best", "rounds": 1, "arith": "auto", "whole": False},
        # the paper's 1-in-3 family at its largest size, 300 variables
        {"name": "cubic1in3-N300", "kind": "count", "family": "cubic1in3", "n": 200, "m": 0, "index": 0,
         "order": "best", "rounds": 1, "arith": "auto", "whole": False},
        # the benchmark's headline formula: 1-in-3, 300 variables, 186 clauses
        {"name": "1in3-n300", "kind": "count", "family": "1in3", "n": 300, "m": 186, "index": 1, "order": "best",
         "rounds": 24, "arith": "auto", "whole": False},
        # a mixed batch of 256 uneven formulas, 30 to 120 variables
        {"name": "batch-256", "kind": "batch", "count": 256, "order": "greedy"},
        # one training step of the scorer: 64 states, as the shipped training
        {"name": "scorer-train-64", "kind": "scorer", "groups": 64, "train": True},
        # scoring the candidate pairs of one state
        {"name": "scorer-forward-1", "kind": "scorer", "groups": 1, "train": False},
    ]


def draw(rng):
    for _ in range(64):
        c = _draw(rng)
        if c["kind"] != "count":
            return c
        # sizes whose order fits the rank cap and the largest listed cost
        try:
            net, plan = _plan(c, 0)
        except tn.TNError:
            continue
        if (2.0 ** plan.stats["log2_cost"] <= MAX_PREDICTED_US
                and tn.workspace_bytes(net, plan, **_count_args(c)) <= MAX_WORKSPACE):
            return c
    raise RuntimeError("no drawable case")


def _draw(rng):
    what = rng.choice(["cvc", "cvc", "1in3", "1in3", "cubic1in3", "3cnf", "hardcore", "primes", "batch", "scorer"])
    index = rng.randrange(1 << 10)
    if what == "batch":
        return {"kind": "batch", "count": int(round(16 * 16 ** rng.random())), "order": "greedy"}
    if what == "scorer":
        return {"kind": "scorer", "groups": int(round(256 ** rng.random())), "train": rng.random() < 0.7}
    arith, m, family = "auto", 0, what
    if what == "cvc":
        n = 2 * int(round(10 * 10 ** rng.random()))
    elif what == "primes":
        n, family, arith = 2 * rng.randint(30, 100), "cvc", "primes"
    elif what == "cubic1in3":
        n = 2 * rng.randint(10, 100)
    elif what == "hardcore":
        n = 2 * rng.randint(10, 70)
    elif what == "3cnf":
        n = rng.randint(20, 60)
        m = int(round(rng.uniform(1.0, 1.2) * n))
    else:
        n = int(round(20 * 15 ** rng.random()))
        m = int(round(rng.uniform(0.60, 0.66) * n))
    return {"kind": "count", "family": family, "n": n, "m": m, "index": index,
            "order": "greedy" if n <= 64 and family in ("cvc", "1in3") else "best",
            "rounds": 0 if n <= 64 and family in ("cvc", "1in3") else 1, "arith": arith,
            "whole": n <= 40 and family in ("cvc", "1in3")}


# ------------------------------------------------------------------ inputs
def _formula(case, seed):
    """The case's formula: the graph from ``index``, the data from ``seed``."""
    fam, n, m, idx = case["family"], case["n"], case["m"], case["index"]
    r = random.Random(1000003 * (seed + 1) + idx)
    if fam == "hardcore":
        # vertex weights of up to 1000
        c = I.hardcore_csp(I.cubic_graph(n, I.Rng(idx)), n, 1000)
        cons = [(scope, [1, r.randint(500, 1000)] if len(scope) == 1 else table) for scope, table in c.constraints]
        return I.CSP(c.n_vars, c.domain, cons, name=c.name)
    if fam == "cvc":
        f, flip = I.cvc(n, idx), 0.5
    elif fam == "cubic1in3":
        f, flip = I.cubic_1in3(n, idx), 1.0 / 16
    elif fam == "3cnf":
        f, flip = I.exactly_one_3(n, m, I.Rng(I.instance_seed(7, idx))), 0.5
        f.clauses = [(I.OR, c) for _, c in f.clauses]
    elif (n, m) == (20, 14):
        f, flip = I.small_1in3(idx), 1.0 / 16
    else:
        f, flip = I.large_1in3(n, m / n, idx), 1.0 / 16
    f.clauses = [(k, [-v if r.random() < flip else v for v in c]) for k, c in f.clauses]
    return f


def _plan(case, seed):
    net = tn.Network(_formula(case, seed))
    return net, net.order(case["order"], case["index"], rounds=case["rounds"])


def _count_args(case):
    # up to 16 residue planes resident together, as a program with the whole
    # GPU to itself asks for
    if case["arith"] == "primes":
        return {"arith": "rns", "flags": tn.FLAG_WIDE_RNS, "prime_group": 16}
    return {"prime_group": 16}


def _batch(case, seed):
    return [I.batch_instance(i, master=seed) for i in range(case["count"])]


def _rows(case, seed):
    """Group offsets of a scorer case: uneven candidate lists."""
    r = np.random.default_rng(case["groups"])
    sizes = r.integers(ROWS_PER_GROUP // 2, 3 * ROWS_PER_GROUP // 2 + 1, size=case["groups"])
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)


def _scorer_data(case, seed):
    """Host arrays of a scorer case: parameters, features (small counts and
    ranks, scaled), labels (one to three merges per state), group offsets and
    Adam's moments after some steps."""
    g = _rows(case, seed)
    n = int(g[-1])
    r = np.random.default_rng(seed)
    x = (r.integers(0, 24, size=(n, FEATURES)) / 8.0).astype(np.float32)
    lab = np.zeros(n, dtype=np.uint8)
    for k in range(case["groups"]):
        lab[r.integers(g[k], g[k + 1], size=1 + k % 3)] = 1
    p = init_params(seed)
    m = r.normal(0, 1e-3, p.size).astype(np.float32)
    v = (r.uniform(0.5, 2.0, p.size) * 1e-4).astype(np.float32)
    return p, x, lab, g, m, v


ADAM_STEP, ADAM_LR = 100, 2e-3


def prepare(case, seed):
    if case["kind"] == "batch":
        return {"case": case, "formulas": _batch(case, seed)}
    if case["kind"] == "scorer":
        p, x, lab, g, m, v = (torch.from_numpy(a).cuda() for a in _scorer_data(case, seed))
        n = x.shape[0]
        f = dict(dtype=torch.float32, device="cuda")
        s = {"case": case, "p": p, "x": x, "lab": lab, "g": g, "m": m, "v": v,
             "h1": torch.empty(n, HIDDEN, **f), "h2": torch.empty(n, HIDDEN, **f), "y": torch.empty(n, **f)}
        if case["train"]:
            s.update(dz1=torch.empty(n, HIDDEN, **f), dz2=torch.empty(n, HIDDEN, **f), dy=torch.empty(n, **f),
                     grad=torch.empty_like(p), loss=torch.empty(1, **f))
        return s
    if case["whole"]:
        return {"case": case, "formula": _formula(case, seed)}
    net, plan = _plan(case, seed)
    return {"case": case, "net": net, "plan": plan, "args": _count_args(case)}


def _limbs(count):
    return np.frombuffer(count.to_bytes(4 * LIMBS, "little"), dtype=np.uint32)


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        return np.stack([_limbs(c) for c in tn.count_batch(state["formulas"], case["order"], seed=0)])
    if case["kind"] == "scorer":
        s = state
        tn.mlp_forward(s["p"], s["x"], s["h1"], s["h2"], s["y"])
        if not case["train"]:
            return {"h1": s["h1"], "h2": s["h2"], "y": s["y"]}
        tn.mlp_backward(s["p"], s["x"], s["h1"], s["h2"], s["y"], s["lab"], s["g"], s["grad"], s["dz2"], s["dz1"],
                        s["dy"], s["loss"])
        tn.mlp_adam(s["p"], s["grad"], s["m"], s["v"], ADAM_STEP, lr=ADAM_LR)
        return {k: s[k] for k in ("y", "loss", "dy", "dz2", "dz1", "grad", "p", "m", "v")}
    if case["whole"]:
        return _limbs(tn.count(state["formula"], case["order"]))
    return _limbs(tn.count_plan(state["net"], state["plan"], **state["args"]))


# -------------------------------------------------------------------- work
def work(case):
    """Counts: along the order in hand, every step reads its two tensors once
    and writes one, in every residue plane (one byte per small modulus, 4
    bytes per 16-bit prime, 8 per 64-bit count), and does one multiply-add
    per term of its sum. Scorer: each tensor that comes in or goes out once."""
    if case["kind"] == "scorer":
        n = int(_rows(case, 0)[-1])
        p = HIDDEN * (FEATURES + 1) + HIDDEN * (HIDDEN + 1) + HIDDEN + 1
        fwd = 2.0 * n * (HIDDEN * FEATURES + HIDDEN * HIDDEN + HIDDEN)
        if not case["train"]:
            return {"bytes": 4.0 * (p + n * (FEATURES + 2 * HIDDEN + 1)), "flops": fwd}
        return {"bytes": 4.0 * (8 * p + n * (FEATURES + 4 * HIDDEN + 2)) + n, "flops": 3.0 * fwd}
    if case["kind"] == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for f in _batch(case, 0):
            net = tn.Network(f)
            for k, v in _count_work(net.order(case["order"], 0), {}).items():
                total[k] += v
        return total
    return _count_work(_plan(case, 0)[1], {k: v for k, v in _count_args(case).items() if k != "prime_group"})


def _count_work(plan, args):
    mods = tn.moduli(plan, **args)
    planes = max(1, len(mods))
    size = 8 if not mods else 1 if max(mods) <= 255 else 4
    return {"bytes": planes * size * plan.stats["entries"], "flops": 2.0 * planes * plan.stats["macs"]}


# ------------------------------------------------------------------- exact
def exact(case, seed):
    """Counts: enumeration of all assignments where there are few. Scorer:
    the same step in float64."""
    if case["kind"] == "count" and case["family"] != "hardcore" and case["n"] <= 22:
        return _limbs(_enumerate(_formula(case, seed)))
    if case["kind"] != "scorer":
        return None
    p, x, lab, g, m, v = (a.astype(np.float64) if a.dtype == np.float32 else a for a in _scorer_data(case, seed))
    H, F = HIDDEN, FEATURES
    cuts = np.cumsum([H * F, H, H * H, H, H])
    w1, b1, w2, b2, w3, b3 = np.split(p, cuts)
    w1, w2 = w1.reshape(H, F), w2.reshape(H, H)
    h1 = np.maximum(x @ w1.T + b1, 0.0)
    h2 = np.maximum(h1 @ w2.T + b2, 0.0)
    y = h2 @ w3 + b3
    if not case["train"]:
        return {"h1": h1, "h2": h2, "y": y}
    groups = len(g) - 1
    dy, loss = np.zeros_like(y), 0.0
    for k in range(groups):
        s = slice(g[k], g[k + 1])
        e = np.exp(y[s] - y[s].max())
        pos = e * (lab[s] > 0)
        loss += (math.log(e.sum()) - math.log(pos.sum())) / groups
        dy[s] = (e / e.sum() - pos / pos.sum()) / groups
    dz2 = dy[:, None] * w3[None, :] * (h2 > 0)
    dz1 = (dz2 @ w2) * (h1 > 0)
    grad = np.concatenate([(dz1.T @ x).ravel(), dz1.sum(0), (dz2.T @ h1).ravel(), dz2.sum(0), h2.T @ dy, [dy.sum()]])
    m = 0.9 * m + 0.1 * grad
    v = 0.999 * v + 0.001 * grad * grad
    p = p - ADAM_LR * (m / (1 - 0.9 ** ADAM_STEP)) / (np.sqrt(v / (1 - 0.999 ** ADAM_STEP)) + 1e-8)
    return {"y": y, "loss": np.array([loss]), "dy": dy, "dz2": dz2, "dz1": dz1, "grad": grad, "p": p, "m": m, "v": v}


def _enumerate(f):
    a = np.arange(1 << f.n_vars, dtype=np.int64)
    ok = np.ones(a.size, dtype=bool)
    for kind, lits in f.clauses:
        t = np.zeros(a.size, dtype=np.int8)
        for v in lits:
            t += (((a >> (abs(v) - 1)) & 1) == (1 if v > 0 else 0)).astype(np.int8)
        ok &= t >= 1 if kind == I.OR else t == 1 if kind == I.EXACTLY_ONE else t % 2 == 1
    return int(ok.sum())
