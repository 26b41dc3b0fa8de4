"""The calls whose time on the GPU counts for a user of this framework.

Two kinds of case, both through the package's public classes:

* ``solve``: one ``Solver``.  A pass runs ``iters`` iterations, evaluates the
  average profile and copies both players' average strategies out: what a
  program does between two reports of a solve.
* ``batch``: one ``Batch`` of ``games`` games of uneven size.  A pass runs
  ``iters`` iterations with a check every ten, reads every game's status and
  copies every game's average strategies out.

Games are public trees with private signals (the generator's family): a
tree's shape belongs to the case, its payoffs come from the seed.  A game
starts at the uniform strategy and every pass continues its solve.

A case's fields: ``depth``, ``branch`` and ``frac`` (every public node has
``branch`` actions or, with probability ``frac``, one more), ``stop`` (a node
ends the game early with that probability), ``signals``, ``payoff`` ("iid":
uniform per terminal and signal pair; "showdown": the sign of the signals'
difference times a pot), ``tree`` (the shape's own seed), ``precision``,
``variant``, ``mode``, ``iters``, and ``quads`` (the product tiling: the
default, or the quad streams that the autotuner keeps on large games, set
once as a program with cached tunings does).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import gamegen as gg
import paper_2605_14277_amd as cfr

QUADS = {"items": [16, 16], "rows": [256, 256], "vec": [3, 3], "perm": [0, 1], "xcd": [1, 1]}


def _solve(name, depth, branch, frac, signals, *, stop=0.0, payoff="iid", tree=1, precision="fp64",
           variant="cfr+", mode="alternating", iters=50, quads=False):
    return {"name": name, "kind": "solve", "depth": depth, "branch": branch, "frac": frac,
            "signals": signals, "stop": stop, "payoff": payoff, "tree": tree,
            "precision": precision, "variant": variant, "mode": mode, "iters": iters,
            "quads": quads}


def listed():
    return [
        # a toy game (16 terminals, 144 nonzeros), solved inside a loop or a
        # test: launches and latency only
        _solve("tiny-vanilla-fp64", 4, 2, 0.0, 3, variant="vanilla", mode="simultaneous",
               iters=200),
        # a research-sized card game (13 signals, early stops, about 5e4
        # nonzeros), the default precision and tiling
        _solve("small-cfrplus-fp64", 8, 2, 0.5, 13, stop=0.15, tree=2000, iters=100),
        # the small end of the showdown games (about 2e5 nonzeros)
        _solve("small-dcfr-acc64", 6, 2, 0.98, 16, payoff="showdown", variant="dcfr",
               precision="fp32_acc64", iters=40),
        # few levels, many actions (9 or 10 a decision point): the sweeps'
        # general code, predictive updates
        _solve("wide-pcfrplus-fp64", 4, 9, 0.6, 12, variant="pcfr+", iters=50),
        # the medium game (depth 13, early stops, 3.4e6 nonzeros) in double
        _solve("medium-cfrplus-fp64", 13, 2, 0.5, 13, stop=0.15, tree=2012, iters=50),
        # a medium game with an odd signal count, all in float, both players
        # moving at once
        _solve("medium-vanilla-fp32", 8, 3, 0.2, 19, variant="vanilla", mode="simultaneous",
               precision="fp32", iters=40),
        # 1e7 nonzeros, quad streams, predictive updates, continuous payoffs
        _solve("mid-pcfrplus-acc64", 8, 3, 0.15, 32, variant="pcfr+", precision="fp32_acc64",
               iters=40, quads=True),
        # the upper-middle showdown game in double (2.4e7 nonzeros)
        _solve("upper-dcfr-fp64", 10, 3, 0.15, 16, payoff="showdown", variant="dcfr", iters=50,
               quads=True),
        # a game of the large benchmark's size (1e5 terminals, 32 signals, about
        # 1e8 nonzeros)
        _solve("large-dcfr-acc64", 10, 3, 0.15, 32, payoff="showdown", variant="dcfr",
               precision="fp32_acc64", iters=100, quads=True),
        # many small games solved together (repeated play, sweeps of
        # parameters), and a batch of uneven ones up to a few 1e6 nonzeros
        {"name": "batch-small", "kind": "batch", "games": 24, "t_lo": 16.0, "t_hi": 300.0,
         "s_hi": 8, "tree": 4000, "precision": "fp32_acc64", "variant": "pcfr+",
         "mode": "alternating", "iters": 40},
        {"name": "batch-uneven", "kind": "batch", "games": 24, "t_lo": 100.0, "t_hi": 10000.0,
         "s_hi": 24, "tree": 4001, "precision": "fp32_acc64", "variant": "dcfr",
         "mode": "alternating", "iters": 40},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    precision = rng.choice(["fp64", "fp32", "fp32_acc64"])
    variant = rng.choice(["vanilla", "cfr+", "dcfr", "pcfr+", "pcfr"])
    mode = rng.choice(["alternating", "alternating", "simultaneous"])
    if rng.random() < 0.2:
        t_hi = _log_uniform(rng, 100, 10000)
        return {"kind": "batch", "games": rng.randint(4, 28), "t_lo": 16.0, "t_hi": t_hi,
                "s_hi": rng.randint(4, 24), "tree": rng.randrange(1 << 20),
                "precision": precision, "variant": variant, "mode": mode,
                "iters": rng.choice([20, 40, 60])}
    signals = rng.randint(3, 32)
    nnz = _log_uniform(rng, 100, 4e7 if precision != "fp64" else 2e7)
    terminals = max(16.0, nnz / signals ** 2)
    depth = rng.randint(max(2, math.ceil(math.log(terminals) / math.log(12.0))),
                        max(2, min(10, math.floor(math.log(terminals) / math.log(2.0)))))
    root = terminals ** (1.0 / depth)
    iters = max(20, min(200 if precision == "fp64" else 40, int(1e9 / nnz)))
    case = _solve("", depth, max(1, int(root)), round(root - int(root), 3), signals,
                  payoff=rng.choice(["iid", "showdown"]), tree=rng.randrange(1 << 20),
                  precision=precision, variant=variant, mode=mode, iters=iters,
                  quads=nnz > 5e6 or rng.random() < 0.25)
    del case["name"]
    return case


# ---- games -----------------------------------------------------------------

class _Game:
    """The arrays a Solver or a Batch takes."""

    def __init__(self, **arrays):
        self.__dict__.update(arrays)

    @property
    def nnz(self):
        return int(self.col_idx.shape[0])


def _shape(depth, branch, frac, stop, tree):
    rng = np.random.Generator(np.random.PCG64(tree))
    if stop:
        return gg.make_public_tree(rng, depth, branch, branch + 1, stop)
    return gg.make_public_tree(rng, depth, branch, branch + 1, 0.0, branch_p_hi=frac)


@functools.lru_cache(maxsize=64)
def _plan(depth, branch, frac, tree, signals):
    """A tree without early stops: both treeplexes, and the rows of both
    products with each row's run of columns, all on the host and small.
    Level l of player p holds the public nodes of depth 2 l + p; its
    sequences are ordered by node, then signal, then action."""
    t = _shape(depth, branch, frac, 0.0, tree)
    S = signals
    nodes = [np.nonzero(t.depth == d)[0] for d in range(depth + 1)]
    k = [t.n_child[n].astype(np.int64) for n in nodes]              # actions of each node
    pos = [np.cumsum(x) - x for x in k]                             # of the nodes before it
    par = [None] + [np.repeat(np.arange(len(k[d])), k[d]) for d in range(depth)]
    act = [None] + [np.arange(len(nodes[d + 1])) - pos[d][par[d + 1]] for d in range(depth)]
    base, n_seq, n_inf, inf_parent, inf_first = [0] * depth, [1, 1], [0, 0], [[], []], [[], []]
    sig = np.arange(S)
    for d in range(depth):
        p = d & 1
        base[d] = n_seq[p]
        inf_first[p].append((base[d] + S * pos[d][:, None] + sig * k[d][:, None]).reshape(-1))
        if d < 2:
            inf_parent[p].append(np.zeros(len(k[d]) * S, np.int64))
        else:
            g = par[d - 1][par[d]]
            a = act[d - 1][par[d]]
            inf_parent[p].append((base[d - 2] + S * pos[d - 2][g][:, None] +
                                  sig * k[d - 2][g][:, None] + a[:, None]).reshape(-1))
        n_seq[p] += S * int(k[d].sum())
        n_inf[p] += S * len(k[d])
    first = [np.concatenate(inf_first[p] + [[n_seq[p]]]).astype(np.int32) for p in range(2)]
    parent = [np.concatenate(inf_parent[p]).astype(np.int32) for p in range(2)]
    # every terminal hangs below the last node of both players: the mover of
    # depth - 1 (m) and of depth - 2 (o)
    m, o = depth - 1, depth - 2
    zfirst = pos[m]
    child = np.arange(len(k[m]))                                    # m's node below (o's node, action)
    rows = {}
    # o's row (node, s, a): the run of all sequences of the node below
    rows[o & 1] = {"lvl": o, "node": np.repeat(par[m], S), "slot": np.tile(sig, len(child)),
                   "start": np.repeat(base[m] + S * pos[m][child], S), "stride": 0,
                   "k": np.repeat(k[m], S), "z": np.repeat(zfirst, S),
                   "row": (base[o] + S * pos[o][par[m]][:, None] + sig * k[o][par[m]][:, None] +
                           act[m][:, None]).reshape(-1)}
    # m's row (node, s, a): one sequence of the node above for every signal
    zn, za = par[depth], act[depth]
    up = par[m][zn]
    rows[m & 1] = {"lvl": m, "slot": np.tile(sig, len(zn)),
                   "start": np.repeat(base[o] + S * pos[o][up] + act[m][zn], S),
                   "stride": np.repeat(k[o][up], S), "k": np.ones(len(zn) * S, np.int64),
                   "z": np.repeat(np.arange(len(zn)), S),
                   "row": (base[m] + S * pos[m][zn][:, None] + sig * k[m][zn][:, None] +
                           za[:, None]).reshape(-1)}
    return n_seq, n_inf, parent, first, rows, len(zn), S


def _products(plan, payoff, values, device):
    """(ptr, idx, val) of A by rows and by columns."""
    n_seq, _, _, _, rows, _, S = plan
    out = []
    for p in range(2):
        r = rows[p]
        order = np.argsort(r["row"], kind="stable")
        up = {f: torch.from_numpy(np.ascontiguousarray(np.broadcast_to(r[f], order.shape)[order]))
              .to(device) for f in ("row", "slot", "start", "stride", "k", "z")}
        length = S * up["k"]
        at = torch.repeat_interleave(length)                        # row of every entry
        j = torch.arange(at.numel(), device=device) - (torch.cumsum(length, 0) - length)[at]
        kk = up["k"][at]
        s_col, a = torch.div(j, kk, rounding_mode="floor"), j % kk
        z = up["z"][at] + a
        col = up["start"][at] + torch.where(up["stride"][at] > 0, s_col * up["stride"][at], j)
        s_row = up["slot"][at]
        s1, s2 = (s_row, s_col) if p == 0 else (s_col, s_row)
        if payoff == "iid":
            val = values[z, s1, s2] / (S * S)
        else:
            val = torch.sign(s1 - s2) * values[z] / (S * S)
        keep = val != 0
        ptr = torch.zeros(n_seq[p] + 1, dtype=torch.int64, device=device)
        ptr[1:] = torch.cumsum(torch.bincount(up["row"][at[keep]], minlength=n_seq[p]), 0)
        out.append((ptr.cpu().numpy(), col[keep].to(torch.int32).cpu().numpy(),
                    val[keep].cpu().numpy()))
    return out


def _game(case, seed):
    rng = np.random.Generator(np.random.PCG64([case["tree"], seed]))
    S = case["signals"]
    if case["stop"] or case["depth"] < 2:
        t = _shape(case["depth"], case["branch"], case["frac"], case["stop"], case["tree"])
        pay = (rng.uniform(-1.0, 1.0, (t.n_terminals, S, S)) if case["payoff"] == "iid"
               else rng.uniform(1.0, 8.0, t.n_terminals))
        return gg.build_game(t, S, S, case["payoff"], pay)
    plan = _plan(case["depth"], case["branch"], case["frac"], case["tree"], S)
    n_seq, n_inf, parent, first, _, T, _ = plan
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    pay = (rng.uniform(-1.0, 1.0, (T, S, S)) if case["payoff"] == "iid"
           else rng.uniform(1.0, 8.0, T))
    (rp, ri, rv), (cp, ci, cv) = _products(plan, case["payoff"],
                                           torch.from_numpy(pay).to(device), device)
    return _Game(n_seq=n_seq, n_inf=n_inf, inf_parent=parent, inf_first_seq=first, row_ptr=rp,
                 col_idx=ri, val=rv, col_ptr=cp, row_idx=ci, val_csc=cv)


def _batch_cases(case):
    """The games of a batch as solve cases: sizes as the generator's batch
    distribution draws them, at this case's limits."""
    specs = gg.batch_specs(case["games"], seed=case["tree"], t_lo=case["t_lo"], t_hi=case["t_hi"],
                           s_hi=case["s_hi"], d_lo=4, d_hi=8)
    return [_solve("", s["depth"], s["branch_lo"], round(s["branch_p_hi"], 3), s["S"],
                   tree=s["seed"], precision=case["precision"], variant=case["variant"],
                   mode=case["mode"], iters=case["iters"]) for s in specs]


# ---- a case on the GPU --------------------------------------------------------

def prepare(case, seed):
    if case["kind"] == "solve":
        solver = cfr.Solver(_game(case, seed), precision=case["precision"])
        if case["quads"]:
            solver.tiling = QUADS
        return {"solver": solver, "iters": case["iters"], "variant": case["variant"],
                "mode": case["mode"]}
    games = [_game(c, seed) for c in _batch_cases(case)]
    sizes = sum(cfr.Batch.game_size(g) for g in games)
    batch = cfr.Batch([int(v) for v in sizes[0:2]], [int(v) for v in sizes[2:4]], int(sizes[4]),
                      max_games=len(games), precision=case["precision"], mode=case["mode"])
    ids = [batch.add(g, case["variant"]) for g in games]
    return {"batch": batch, "ids": ids, "iters": case["iters"]}


def run(state):
    if "solver" in state:
        s = state["solver"]
        s.step(state["iters"], state["variant"], state["mode"])
        e = s.exploitability("average")
        return {"profile": [e["expl"], e["nash_conv"], e["br1"], e["br2"], e["value"]],
                "average": [s.strategy(p, "average") for p in range(2)]}
    b = state["batch"]
    b.run(state["iters"])
    return {"expl": np.array([b.status(g)["expl"] for g in state["ids"]]),
            "average": [b.strategy(g, p, "average") for g in state["ids"] for p in range(2)]}


# ---- what a pass cannot do without ----------------------------------------------

def _sizes(case):
    """(nonzeros, sequences of both players) of a solve case's game."""
    S = case["signals"]
    if not case["stop"] and case["depth"] >= 2:
        n_seq, _, _, _, _, T, _ = _plan(case["depth"], case["branch"], case["frac"], case["tree"], S)
        n = sum(n_seq)
    else:
        t = _shape(case["depth"], case["branch"], case["frac"], case["stop"], case["tree"])
        T, n = t.n_terminals, S * (t.n_nodes - 1) + 2
    return T * S * (S - 1 if case["payoff"] == "showdown" else S), n


def work(case):
    """Per iteration the payoffs once for either product with one column each,
    and per sequence its utility and strategies and the regret and average
    accumulators read and written; then the evaluation's two products and the
    strategies that leave."""
    cases = [case] if case["kind"] == "solve" else _batch_cases(case)
    v = 8 if case["precision"] == "fp64" else 4
    a = 4 if case["precision"] == "fp32" else 8
    checks = 1 if case["kind"] == "solve" else case["iters"] // 10
    total = {"bytes": 0.0, "flops": 0.0}
    for c in cases:
        nnz, n = _sizes(c)
        it = 2 * nnz * (4 + v) + n * (4 * v + 4 * a + 4)
        total["bytes"] += case["iters"] * it + checks * 2 * nnz * (4 + v) + 8 * n
        total["flops"] += (case["iters"] + checks) * (4 * nnz + 12 * n)
    return total


# ---- the same in 64 bits -------------------------------------------------------

class _Player:
    def __init__(self, n_seq, parent, first, sign):
        self.n, self.sign = int(n_seq), sign
        parent, first = np.asarray(parent, np.int64), np.asarray(first, np.int64)
        count = np.diff(first)
        self.inf = np.zeros(self.n, np.int64)                       # decision point of a sequence
        self.inf[1:] = np.repeat(np.arange(len(parent)), count)
        self.up = np.zeros(self.n, np.int64)
        self.up[1:] = np.repeat(parent, count)
        self.parent, self.width = parent, count
        level = np.zeros(len(parent), np.int64)
        while True:                                                 # own decisions before it
            deeper = np.where(parent > 0, level[self.inf[parent]] + 1, 0)
            if np.array_equal(deeper, level):
                break
            level = deeper
        self.levels = []
        for lv in range(int(level.max()) + 1 if len(level) else 0):
            js = np.nonzero(level == lv)[0]
            seqs = np.nonzero(np.isin(level[self.inf[1:]], lv))[0] + 1
            self.levels.append((js, seqs))
        self.r, self.m, self.s = np.zeros(self.n), np.zeros(self.n), np.zeros(self.n)
        self.b = np.ones(self.n)
        self.match(self.r)
        self.x = np.ones(self.n)
        self.down()

    def match(self, r):
        z = np.maximum(r, 0.0)
        total = np.bincount(self.inf[1:], z[1:], minlength=len(self.parent))[self.inf[1:]]
        self.b[1:] = np.where(total > 0, z[1:] / np.where(total > 0, total, 1.0),
                              1.0 / self.width[self.inf[1:]])

    def down(self):
        self.x[0] = 1.0
        for _, seqs in self.levels:
            self.x[seqs] = self.x[self.up[seqs]] * self.b[seqs]

    def values(self, g, best=False):
        """Counterfactual value of every sequence and decision point, and at
        the empty sequence."""
        q = self.sign * g
        v = np.full(len(self.parent), -np.inf) if best else np.zeros(len(self.parent))
        for js, seqs in reversed(self.levels):
            if best:
                np.maximum.at(v, self.inf[seqs], q[seqs])
            else:
                v += np.bincount(self.inf[seqs], self.b[seqs] * q[seqs], minlength=len(v))
            np.add.at(q, self.parent[js], v[js])
        return q, v

    def observe(self, g, variant, t):
        q, v = self.values(g)
        inst = np.zeros(self.n)
        inst[1:] = q[1:] - v[self.inf[1:]]
        r = self.r + inst
        if variant in ("cfr+", "pcfr+"):
            r = np.maximum(r, 0.0)
        elif variant == "dcfr":
            r = np.where(r > 0, r * (t ** 1.5 / (t ** 1.5 + 1.0)), r * 0.5)
        self.r = r
        self.match(r + inst if variant.startswith("pcfr") else r)

    def move(self, w):
        self.s += w * self.x
        self.down()


def _exact_solve(case, seed):
    g = _game(case, seed)
    rows = np.repeat(np.arange(g.n_seq[0]), np.diff(g.row_ptr))
    cols, val = np.asarray(g.col_idx, np.int64), np.asarray(g.val, np.float64)
    one, two = (_Player(g.n_seq[p], g.inf_parent[p], g.inf_first_seq[p], (1.0, -1.0)[p])
                for p in range(2))

    def ay(y):
        return np.bincount(rows, val * y[cols], minlength=g.n_seq[0])

    def atx(x):
        return np.bincount(cols, val * x[rows], minlength=g.n_seq[1])

    variant, total = case["variant"], 0.0
    for t in range(1, case["iters"] + 1):
        w = {"cfr+": float(t), "dcfr": float(t) ** 2, "pcfr+": float(t) ** 2}.get(variant, 1.0)
        total += w
        g1 = ay(two.x)
        g2 = atx(one.x) if case["mode"] == "simultaneous" else None
        one.observe(g1, variant, t)
        one.move(w)
        two.observe(atx(one.x) if g2 is None else g2, variant, t)
        two.move(w)
    x, y = one.s / total, two.s / total
    x[0] = y[0] = 1.0
    best1, best2 = one.values(ay(y), best=True)[0][0], two.values(atx(x), best=True)[0][0]
    profile = [(best1 + best2) / 2.0, best1 + best2, best1, best2, float(x @ ay(y))]
    return [np.float64(v) for v in profile], [x, y]


def exact(case, seed):
    """Plain numpy in double: the iterations of the paper's Algorithm 2 with
    the variant's update, decision points level by level.  Only for games
    where that takes seconds; in float the trajectory of a long solve parts
    from it by itself, and so does that of a showdown game, where regrets
    that are exactly zero by symmetry decide strategies by their rounding:
    those have no such value either."""
    cases = [case] if case["kind"] == "solve" else _batch_cases(case)
    cost = sum(_sizes(c)[0] + 3 * _sizes(c)[1] for c in cases) * case["iters"]
    if cost > 5e8:
        return None
    if case["precision"] != "fp64" and (case["iters"] > 40 or case.get("payoff") == "showdown"):
        return None
    got = [_exact_solve(c, seed) for c in cases]
    if case["kind"] == "solve":
        return {"profile": got[0][0], "average": got[0][1]}
    return {"expl": np.array([p[0] for p, _ in got]), "average": [v for _, s in got for v in s]}
