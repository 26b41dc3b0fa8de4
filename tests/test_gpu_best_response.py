"""Best-response values where the shallow levels' launch begins and ends: a
level of 1024 decision points of a game is its last to fit, 24 levels are its
most, and the decision points below the empty sequence are summed 1024 at a
time; alone and in a batch, against the oracle, to the 1e-9 that
FP64 is held to (a level left out or taken early moves them by far more)."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


def chain(depth):
    return gg.public_game(3, S=2, max_depth=depth, branch_lo=1, branch_hi=1, p_stop=0.0)


def wide(S, depth):
    return gg.public_game(3, S=S, max_depth=depth, branch_lo=1, branch_hi=2, p_stop=0.0)


# max_depth d gives each player d / 2 levels
GAMES = {"points-1024": lambda: wide(1024, 3), "points-1025": lambda: wide(1025, 3),
         "levels-24": lambda: chain(48), "levels-25": lambda: chain(50),
         "fewer": gg.cfg1}


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


def values(e):
    return [float(e[k]) for k in ("expl", "nash_conv", "br1", "br2")]


def same(got, want):
    return np.all(np.abs(np.subtract(got, want)) <= 1e-9 * np.maximum(1.0, np.abs(want)))


def test_values_are_the_oracles(cfr, oracle_mod):
    games = {n: f() for n, f in GAMES.items()}
    size = sum(cfr.Batch.game_size(g) for g in games.values())
    b = cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                  max_games=len(games), precision="fp64")
    ids = {n: b.add(g, "cfr+") for n, g in games.items()}
    b.run(20)
    for n, g in games.items():
        o = oracle_mod.Oracle(g)
        s = cfr.Solver(g, precision="fp64")
        o.step(20, "cfr+", "alternating")
        s.step(20, "cfr+", "alternating")
        for kind in ("current", "average"):
            want = values(o.exploitability(kind))
            assert same(values(s.exploitability(kind)), want), (n, kind)
            assert same(values(b.exploitability(ids[n], kind)), want), (n, kind)
        s.close()
    # all of them in one evaluation
    b.run(10)
    for n, g in games.items():
        o = oracle_mod.Oracle(g)
        o.step(30, "cfr+", "alternating")
        assert same(b.status(ids[n])["expl"], o.exploitability("average")["expl"]), n
    b.close()
