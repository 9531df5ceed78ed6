"""The work that users of the evaluator have it do, as cases that can be timed.

Each case is one call of a public entry point on a population over a case matrix.  The listed ones are the shapes
of the benchmark's workloads (bench.py) and what surrounds them: a population of a small run, one generation of a run
evaluated from host arrays, the large resident populations (regression over the full and the arithmetic function set,
classification, the 20-multiplexer, register programs), many populations in one batched launch, per-case predictions,
and odd sizes in between.  `draw` gives other sizes, function sets and fitness kinds of the same ranges.

Programs are size-targeted random trees (PTC2) and uniform random register programs, as in the benchmark.
"""
import math

import numpy as np
import torch

import paper_1601_00221_amd as gp

ADD, SUB, MUL, PDIV, SIN, COS, EXPC, PLOG, AND, OR, NAND, NOR, GT, LT, EQ, IF = range(16)
VAR, CONST = 64, 65
ARITY = np.array([2, 2, 2, 2, 1, 1, 1, 1, 2, 2, 2, 2, 2, 2, 2, 3])
SETS = {
    "arith": (ADD, SUB, MUL),
    "basic": (ADD, SUB, MUL, PDIV),
    "trig": (ADD, SUB, MUL, SIN, COS),
    "full": (ADD, SUB, MUL, PDIV, SIN, COS, EXPC, PLOG),
    "class": (MUL, PDIV, ADD, SUB, GT, LT, EQ, AND, OR, IF),
    "class_full": (ADD, SUB, MUL, PDIV, GT, LT, EQ, AND, OR, IF, SIN, COS, PLOG, EXPC),
    "bool": (AND, OR, NAND, NOR),
}


def listed():
    return [
        # a small run's population on a small table: launches and latency are all there is
        {"name": "tiny", "path": "resident", "form": "tree", "set": "basic", "prog": 100, "cases": 1024, "feat": 1,
         "sizes": "uniform", "max": 64, "kind": "sum_abs"},
        # one generation of a symbolic regression run (population 1000, 100,000 cases), from host arrays: programs
        # are new in every generation, so lowering and upload are part of the call
        {"name": "generation", "path": "oneshot", "form": "tree", "set": "basic", "prog": 1000, "cases": 100000,
         "feat": 1, "sizes": "lognormal", "max": 1000, "kind": "mse"},
        # register programs with constants on a medium table, from host arrays; most sources are registers, as in
        # programs that selection has made use their earlier results
        {"name": "linear_generation", "path": "oneshot", "form": "linear", "set": "basic", "prog": 500, "cases": 20011,
         "feat": 8, "sizes": "uniform", "max": 256, "const": 2, "chain": 0.75, "kind": "mse"},
        # odd sizes between the extremes: a population and a table of no round number
        {"name": "ragged", "path": "resident", "form": "tree", "set": "full", "prog": 333, "cases": 10007, "feat": 5,
         "sizes": "uniform", "max": 200, "kind": "sum_abs"},
        # the headline shape: regression over the full function set
        {"name": "regression", "path": "resident", "form": "tree", "set": "full", "prog": 4096, "cases": 65536,
         "feat": 8, "sizes": "uniform", "max": 256, "kind": "mse"},
        # the same over {+, -, *}: bound by the interpreter, not by the functions
        {"name": "arith", "path": "resident", "form": "tree", "set": "arith", "prog": 4096, "cases": 65536, "feat": 8,
         "sizes": "uniform", "max": 256, "kind": "mse"},
        # register programs over a million cases, counted hits; sources uniform (a first, random population)
        {"name": "linear", "path": "resident", "form": "linear", "set": "basic", "prog": 4096, "cases": 1 << 20,
         "feat": 16, "sizes": "uniform", "max": 256, "const": 0, "chain": 0.0, "kind": "hits"},
        # classification over few inputs (the Shuttle shape)
        {"name": "classes", "path": "resident", "form": "tree", "set": "class", "prog": 4096, "cases": 58000, "feat": 9,
         "sizes": "uniform", "max": 256, "kind": "class_err"},
        # classification over many inputs with every function (the KDD Cup 99 shape): the largest table
        {"name": "classes_wide", "path": "resident", "form": "tree", "set": "class_full", "prog": 4096, "cases": 494021,
         "feat": 41, "sizes": "uniform", "max": 256, "kind": "class_err"},
        # sub-machine-code evaluation: the 20-multiplexer, 32 cases to a word
        {"name": "multiplexer", "path": "resident", "form": "bool", "set": "bool", "prog": 4096, "cases": 1 << 20,
         "feat": 20, "sizes": "uniform", "max": 256, "kind": "hits"},
        # forty populations, trees and register programs, over three tables in one batched launch
        {"name": "batch", "path": "batch", "form": "mixed", "set": "full", "prog": 10000, "cases": 1 << 20, "feat": 8,
         "sizes": "lognormal", "max": 1024, "jobs": 40, "kind": "mse"},
        # the outputs themselves, for every case: predictions of a set of evolved models
        {"name": "predict", "path": "resident", "form": "tree", "set": "trig", "prog": 256, "cases": 65537, "feat": 6,
         "sizes": "uniform", "max": 48, "kind": "cases"},
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    form = rng.choice(["tree", "tree", "tree", "linear", "bool", "class", "class", "predict", "batch"])
    path = rng.choice(["resident", "resident", "oneshot"])
    prog, cases = _spread(rng, 50, 4096), _spread(rng, 1000, 1 << 19)
    c = {"path": path, "form": "tree", "set": "full", "prog": prog, "cases": cases, "feat": rng.randint(1, 12),
         "sizes": rng.choice(["uniform", "lognormal"]), "max": _spread(rng, 32, 512), "kind": "mse"}
    if form == "tree":
        c["set"] = rng.choice(["arith", "basic", "trig", "full"])
        c["kind"] = rng.choice(["mse", "sum_abs", "hits"])
    elif form == "linear":
        c.update(form="linear", set=rng.choice(["basic", "full"]), feat=rng.randint(1, 24), const=rng.choice([0, 2, 5]),
                 chain=rng.choice([0.0, 0.5, 0.75]), kind=rng.choice(["mse", "hits"]))
    elif form == "bool":
        c.update(form="bool", set="bool", feat=rng.randint(6, 24), cases=_spread(rng, 2000, 1 << 22), kind="hits")
    elif form == "class":
        c.update(set=rng.choice(["class", "class_full"]), feat=rng.randint(4, 41), kind="class_err")
    elif form == "predict":
        c.update(path="resident", prog=_spread(rng, 20, 400), cases=_spread(rng, 1000, 70000),
                 set=rng.choice(["arith", "trig"]), max=48, kind="cases")
    else:
        c.update(path="batch", form="mixed", prog=_spread(rng, 400, 4000), jobs=rng.randint(3, 16), sizes="lognormal")
    # no drawn case has more operations than the largest listed one of its kind
    budget = 2.5e11 if c["form"] != "bool" else 5e11
    while c["prog"] * c["cases"] * c["max"] / 2 > budget:
        c["cases"] = c["cases"] * 2 // 3 + 1
    return c


# ---------------------------------------------------------------------------
# Programs
# ---------------------------------------------------------------------------
def _sizes(rng, c, n):
    if c["sizes"] == "lognormal":
        return np.clip(np.rint(rng.lognormal(math.log(64.0), 1.0, n)), 8, c["max"]).astype(np.int64)
    lo = 32 if c["form"] == "linear" and c["max"] > 64 else 1
    return rng.integers(lo, c["max"] + 1, n)


def _trees(rng, sizes, fset, n_feat, p_const, crange):
    """PTC2 trees of the given target sizes, all grown side by side: (tok, cst, off), prefix order."""
    P, M = len(sizes), int(max(sizes))
    fset = np.array(sorted(fset, key=lambda g: ARITY[g]))
    far = ARITY[fset]
    n_le = np.array([int(np.sum(far <= r)) for r in range(4)])          # functions of at most that arity
    rows = np.arange(P)
    op = np.full((P, M), -1, np.int32)
    kid = np.full((P, M, 3), -1, np.int32)
    slot = np.zeros((P, M + 3), np.int32)                               # open argument slots: 4 * parent + position
    nf, n_open = np.zeros(P, np.int64), np.ones(P, np.int64)            # functions so far; the root is an open slot
    slot[:, 0] = -1
    while True:
        left = sizes - nf - n_open                                      # nodes that may still be added
        k = n_le[np.clip(left, 0, 3)]
        act = np.flatnonzero(k > 0)
        if not len(act):
            break
        g = (rng.random(len(act)) * k[act]).astype(np.int64)
        j = (rng.random(len(act)) * n_open[act]).astype(np.int64)
        s, i = slot[act, j], nf[act]
        slot[act, j] = slot[act, n_open[act] - 1]
        n_open[act] -= 1
        op[act, i] = fset[g]
        inner = s >= 0
        kid[act[inner], s[inner] >> 2, s[inner] & 3] = i[inner]
        for a in range(3):
            m = far[g] > a
            slot[act[m], n_open[act[m]]] = 4 * i[m] + a
            n_open[act[m]] += 1
        nf[act] += 1
    # subtree sizes and prefix positions, function by function over all programs
    F = max(1, int(nf.max()))
    size = np.ones((P, F), np.int64)
    for i in range(F - 1, -1, -1):
        has = op[:, i] >= 0
        tot = np.ones(P, np.int64)
        for a in range(3):
            w = has & (ARITY[np.maximum(op[:, i], 0)] > a)
            kk = kid[:, i, a]
            tot += np.where(w, np.where(kk >= 0, size[rows, np.maximum(kk, 0)], 1), 0)
        size[:, i] = tot
    n = np.where(nf > 0, size[:, 0], 1)
    off = np.zeros(P + 1, np.int64)
    np.cumsum(n, out=off[1:])
    tok = np.full(off[-1], -1, np.int32)
    pos = np.zeros((P, F), np.int64)
    for i in range(F):
        has = np.flatnonzero(op[:, i] >= 0)
        if not len(has):
            break
        tok[off[has] + pos[has, i]] = op[has, i]
        at = pos[has, i] + 1
        for a in range(3):
            kk = kid[has, i, a]
            inner = kk >= 0
            pos[has[inner], kk[inner]] = at[inner]
            at = at + np.where(inner, size[has, np.maximum(kk, 0)], 1)
    t = np.flatnonzero(tok < 0)
    is_c = rng.random(len(t)) < p_const
    tok[t] = np.where(is_c, CONST, VAR | (rng.integers(0, n_feat, len(t)) << 8))
    cst = np.zeros(len(tok), np.float32)
    cst[t] = np.where(is_c, rng.uniform(crange[0], crange[1], len(t)), 0.0)
    return tok, cst, off


def _registers(rng, lengths, ops, n_feat, n_const, chain):
    """Register programs: destinations uniform over 8 registers; a source is a register with probability `chain`,
    otherwise uniform over registers, features and constants."""
    off = np.zeros(len(lengths) + 1, np.int64)
    np.cumsum(lengths, out=off[1:])
    L = int(off[-1])
    src = rng.integers(0, 8 + n_feat + n_const, (2, L))
    src = np.where(rng.random((2, L)) < chain, rng.integers(0, 8, (2, L)), src)
    src = np.where(src >= 8 + n_feat, src - (8 + n_feat) + 128, src)
    code = np.array(ops)[rng.integers(0, len(ops), L)] | (rng.integers(0, 8, L) << 8) | (src[0] << 16) | (src[1] << 24)
    cst = rng.uniform(-1.0, 1.0, len(lengths) * n_const).astype(np.float32)
    return code.astype(np.uint32), off, cst, np.arange(len(lengths) + 1, dtype=np.int64) * n_const


def _population(rng, c, n=None, form=None):
    n, form = n or c["prog"], form or c["form"]
    sizes = _sizes(rng, c, n)
    if form == "linear":
        ops = SETS["basic"] if c["form"] == "mixed" else SETS[c["set"]]
        return _registers(rng, sizes, ops, c["feat"], c.get("const", 2), c.get("chain", 0.0))
    p_const, crange = 1.0 / (c["feat"] + 1), (-1.0, 1.0)
    if c["set"] == "class":
        crange = (-200.0, 200.0)
    elif c["set"] == "class_full":
        crange = (-20000.0, 20000.0)
    elif c["set"] == "bool":
        p_const = 0.0
    return _trees(rng, sizes, SETS[c["set"]], c["feat"], p_const, crange)


# ---------------------------------------------------------------------------
# Tables
# ---------------------------------------------------------------------------
def _table(c, seed, cases=None):
    """(X, y) on the GPU: measurements and a target as the function set has them."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    F, N = c["feat"], cases or c["cases"]
    rand = lambda *s: torch.rand(*s, device="cuda", generator=g)  # noqa: E731
    randn = lambda *s: torch.randn(*s, device="cuda", generator=g)  # noqa: E731
    if c["form"] == "bool":
        W = (N + 31) // 32
        X = torch.randint(-(1 << 31), 1 << 31, (F, W), device="cuda", generator=g, dtype=torch.int64).to(torch.int32)
        a, b, s = X[0], X[1 % F], X[F - 1]
        return X, (a & s) | (b & ~s)
    if c["kind"] == "class_err":
        # integer-valued inputs scattered round a centre for each class, most cases in one class
        k = 10 if c["set"] == "class" else 22
        y = torch.multinomial(torch.tensor([0.75] + [0.25 / (k - 1)] * (k - 1), device="cuda"), N, replacement=True,
                              generator=g)
        centre = rand(k, F) * 200 - 100
        X = torch.empty(F, N, device="cuda")
        for f in range(F):
            X[f] = torch.round(centre[y, f] + 15 * randn(N))
        return X, y.float()
    if c["kind"] == "hits":
        X = randn(F, N)
        return X, torch.where((randn(F, 1) * X).sum(0) > 0, 1.0, -1.0)
    span = 1.0 if F == 1 else 5.0
    X = (2 * rand(F, N) - 1) * span
    y = X[0] ** 6 - 2 * X[0] ** 4 + X[0] ** 2 if F == 1 else X[0] * X[1] + 3 * torch.sin(X[-1]) - 0.5 * X[F // 2]
    return X, y + 0.01 * randn(N)


def _out(c, prog, cases):
    return gp.out_tensor("hits" if c["form"] == "bool" else c["kind"], prog, cases)


class _Pop:
    """Program arrays as gp.make_job takes them."""

    def __init__(self, form, arrays):
        if form == "linear":
            self.code, self.off, self.cst, self.cst_off = arrays
            self.n_reg = 8
        else:
            self.tok, self.cst, self.off = arrays
        self.n_prog = len(self.off) - 1


def prepare(c, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    st = {"case": c}
    if c["path"] == "batch":
        tables = [_table(c, seed * 8 + k, n) for k, n in enumerate(_batch_tables(c))]
        per, jobs, outs = c["prog"] // c["jobs"], [], []
        for j, at in enumerate(_batch_places(c)):
            form = "tree" if j % 2 == 0 else "linear"
            outs.append(_out(c, per, 0))
            jobs.append(gp.make_job(_Pop(form, _population(rng, c, per, form)), at, c["kind"], outs[-1]))
        st.update(tables=tables, jobs=jobs, outs=outs)
        return st
    pop = _population(rng, c)
    X, y = _table(c, seed)
    st.update(X=X, y=None if c["kind"] == "cases" else y, out=_out(c, c["prog"], c["cases"]), pop=pop)
    if c["path"] == "resident":
        if c["form"] == "tree":
            st["set"] = gp.ProgSet.tree(*pop, c["feat"])
        elif c["form"] == "bool":
            st["set"] = gp.ProgSet.boolean(pop[0], pop[2], c["feat"])
        else:
            st["set"] = gp.ProgSet.linear(*pop, 8, c["feat"])
    return st


def _batch_tables(c):
    return [max(500, c["cases"] >> 8), max(500, c["cases"] >> 4), c["cases"]]


def _batch_places(c):
    """The table that each population of a batch is evaluated on."""
    return [int(v) for v in np.random.Generator(np.random.PCG64(4)).integers(0, 3, c["jobs"])]


def run(st):
    c = st["case"]
    if c["path"] == "batch":
        gp.gp_eval_batch(st["tables"], st["jobs"])
        return st["outs"]
    if c["path"] == "resident":
        st["set"].eval(st["X"], st["y"], c["kind"], st["out"], n_cases=c["cases"])
    elif c["form"] == "tree":
        gp.gp_eval_tree(*st["pop"], st["X"], st["y"], c["kind"], st["out"])
    elif c["form"] == "bool":
        gp.gp_eval_bool(st["pop"][0], st["pop"][2], st["X"], st["y"], c["kind"], st["out"], c["cases"])
    else:
        gp.gp_eval_linear(*st["pop"], 8, st["X"], st["y"], c["kind"], st["out"])
    return st["out"]


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _mean_size(c, form):
    return float(np.mean(_sizes(np.random.Generator(np.random.PCG64(0)), dict(c, form=form), 4096)))


def _needed(c):
    """Mean number of a register program's instructions that its result depends on."""
    rng = np.random.Generator(np.random.PCG64(0))
    form = dict(c, form="linear")
    code, off, _, _ = _registers(rng, _sizes(rng, form, 200), SETS["basic"], c["feat"], c.get("const", 2),
                                 c.get("chain", 0.0))
    total = 0
    for p in range(200):
        live = {0}
        for w in code[off[p]:off[p + 1]][::-1].tolist():
            if w >> 8 & 255 in live:
                live.discard(w >> 8 & 255)
                live.update(s for s in (w >> 16 & 255, w >> 24) if s < 8)
                total += 1
    return total / 200


def work(c):
    """Each table and program read once and each output written once; one operation a tree node or needed instruction
    and case (a word's 32 cases are one operation)."""
    if c["path"] == "batch":
        tree, lin, per = _mean_size(c, "tree"), _needed(c), c["prog"] // c["jobs"]
        tables = _batch_tables(c)
        ops = sum(per * tables[at] * (tree if j % 2 == 0 else lin) for j, at in enumerate(_batch_places(c)))
        return {"bytes": 4 * (c["feat"] + 1) * sum(tables) + 8 * c["prog"] * tree + 4 * c["prog"], "flops": ops}
    size = _needed(c) if c["form"] == "linear" else _mean_size(c, c["form"])
    cells = (c["cases"] + 31) // 32 if c["form"] == "bool" else c["cases"]
    out = 4 * c["prog"] * (c["cases"] if c["kind"] == "cases" else 1)
    return {"bytes": 4 * (c["feat"] + 1) * cells + 8 * c["prog"] * size + out, "flops": c["prog"] * cells * size}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
def _apply(op, a, b=None):
    if op == ADD:
        return a + b
    if op == SUB:
        return a - b
    if op == MUL:
        return a * b
    if op == PDIV:
        return torch.where(b.abs() < 1e-6, torch.ones_like(a * b), a / b)
    if op == SIN:
        return torch.sin(a)
    if op == COS:
        return torch.cos(a)
    if op == EXPC:
        return torch.exp(torch.clamp(a, max=88.0))
    return torch.where(a.abs() < 1e-6, torch.zeros_like(a), torch.log(a.abs()))


def exact(c, seed):
    """Trees over the arithmetic and trigonometric sets, node by node in 64 bits.  Whole numbers (hits, classes) have
    no other value, and populations with division, exp or log turn a last place into another result (a protected
    denominator, an overflow of 32 bits), so for those 64 bits say nothing; the batch is made of such populations."""
    if c["form"] != "tree" or c["path"] == "batch" or c["kind"] not in ("mse", "sum_abs", "cases"):
        return None
    if c["set"] not in ("arith", "trig"):
        return None
    tok, cst, off = _population(np.random.Generator(np.random.PCG64(seed)), c)
    X, y = _table(c, seed)
    X, y = X.double(), y.double()
    consts = torch.from_numpy(cst).cuda().double()
    rows = []
    for p in range(c["prog"]):
        stack = []
        for i in range(int(off[p + 1]) - 1, int(off[p]) - 1, -1):      # prefix order backwards: operands come first
            op = int(tok[i]) & 255
            if op == VAR:
                stack.append(X[int(tok[i]) >> 8])
            elif op == CONST:
                stack.append(consts[i])
            elif ARITY[op] == 1:
                stack.append(_apply(op, stack.pop()))
            else:
                a = stack.pop()
                stack.append(_apply(op, a, stack.pop()))
        o = stack.pop().expand(c["cases"])
        if c["kind"] == "cases":
            rows.append(o.clone())
        else:
            d = o - y
            rows.append((d * d).mean() if c["kind"] == "mse" else d.abs().sum())
    return torch.stack(rows)
