"""The resident loop (whole iterations inside one launch) against the launch
per step: the complete state of a solver, and a batch's results, bit for bit.

Every sum is taken in the same order by both, so the comparison is exact.  A
solver with ``use_graph=False`` launches every step; a default one moves to
the resident loop once it has been asked for enough iterations."""
import numpy as np
import pytest

import gamegen as gg
from helpers import dfs_renumber

pytestmark = pytest.mark.gpu

QUADS = {"items": [16, 16], "rows": [256, 256], "vec": [3, 3], "perm": [0, 1], "xcd": [1, 1]}
SMALL = {"items": [4, 8], "rows": [64, 128], "vec": [0, 2], "perm": [1, 1], "xcd": [0, 1]}

GAMES = {
    # one workgroup of 256 threads; of 1024
    "tiny": gg.cfg1,
    "matrix": lambda: gg.matrix_game(np.random.default_rng(1).normal(size=(40, 7))),
    "one-group": lambda: gg.public_game(6, S=5, max_depth=6, branch_lo=2, branch_hi=3, p_stop=0.2),
    # several workgroups on one XCD, without and with a shallow part; early
    # stops leave payoff rows at every level
    "d8": gg.cfg2_literal,
    "deep": lambda: gg.public_game(12, S=3, max_depth=15, branch_lo=1, branch_hi=2, p_stop=0.02),
    # over four actions and over four decision points below one; 64 and more
    "wide": lambda: gg.public_game(8, S=2, max_depth=3, branch_lo=9, branch_hi=12, p_stop=0.0),
    "actions-64": lambda: gg.matrix_game(np.random.default_rng(2).normal(size=(64, 3))),
    "actions-65": lambda: gg.matrix_game(np.random.default_rng(2).normal(size=(65, 3))),
    # rows longer than a chunk; empty rows; a numbering that is permuted
    "long-rows": lambda: gg.public_game(9, S=150, max_depth=2, branch_lo=3, branch_hi=4, p_stop=0.0),
    "showdown": lambda: gg.public_game(4, S=6, max_depth=6, branch_lo=2, branch_hi=4, p_stop=0.1,
                                       payoff_kind="showdown"),
    "depth-first": lambda: dfs_renumber(gg.public_game(5, S=4, max_depth=6, branch_lo=2,
                                                       branch_hi=3, p_stop=0.2)),
    # all compute units
    "units": lambda: gg.public_game(10, S=20, max_depth=8, branch_lo=3, branch_hi=3, p_stop=0.05),
}


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


@pytest.mark.parametrize("precision,variant,mode,tiling", [
    ("fp64", "cfr+", "alternating", None),
    ("fp64", "dcfr", "simultaneous", QUADS),
    ("fp32", "pcfr+", "alternating", SMALL),
    ("fp32_acc64", "pcfr", "alternating", QUADS),
    ("fp32_acc64", "vanilla", "simultaneous", None),
])
@pytest.mark.parametrize("name", list(GAMES))
def test_state_equals_a_launch_per_step(cfr, name, precision, variant, mode, tiling):
    game = GAMES[name]()
    a = cfr.Solver(game, precision=precision)
    b = cfr.Solver(game, precision=precision, use_graph=False)
    for s in (a, b):
        if tiling:
            s.tiling = tiling
    # long enough to be set up, then between other calls; one iteration alone
    # goes the other way
    for n in (600 if name == "units" else 150, 1, 7):
        for s in (a, b):
            s.step(n, variant, mode)
        assert a.exploitability("average") == b.exploitability("average")
        assert a.get_state() == b.get_state()
    # a restored state goes on the same
    image = b.get_state()
    b.step(20, variant, mode)
    a.step(3, variant, mode)
    a.set_state(image)
    a.step(20, variant, mode)
    assert a.get_state() == b.get_state()
    # a new tiling is taken up
    for s in (a, b):
        s.tiling = SMALL if tiling is not SMALL else QUADS
        s.step(300 if name == "units" else 120, variant, mode)
    assert a.get_state() == b.get_state()
    a.close()
    b.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64"])
def test_batches_equal_a_launch_per_step(cfr, precision):
    """Teams of one and of several workgroups side by side, games of
    different variants, one of them stopping early."""
    names = ["tiny", "one-group", "wide", "showdown", "depth-first", "d8"]
    games = [GAMES[n]() for n in names]
    sizes = sum(cfr.Batch.game_size(g) for g in games)
    out = []
    for graph in (True, False):
        b = cfr.Batch([int(v) for v in sizes[:2]], [int(v) for v in sizes[2:4]], int(sizes[4]),
                      max_games=len(games), precision=precision, use_graph=graph)
        ids = [b.add(g, v, max_iterations=m) for g, v, m in
               zip(games, ["cfr+", "dcfr", "pcfr+", "vanilla", "pcfr", "cfr+"],
                   [0, 0, 200, 0, 0, 0])]
        b.run(400)
        out.append([(b.status(i), b.exploitability(i),
                     [b.strategy(i, p, k) for p in range(2) for k in ("current", "average")])
                    for i in ids])
        b.close()
    for x, y in zip(*out):
        assert x[0] == y[0] and x[1] == y[1]
        assert all(np.array_equal(u, v) for u, v in zip(x[2], y[2]))
