"""When the resident loop is set up: after as many iterations as repay it,
counted since the last set-up, so a game that joins a long-lived batch is not
planned for a few of them."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


def small():
    """17,000 sequences: a set-up takes 2.6 to 4.7 ms, 170 to 310 iterations' savings."""
    return gg.public_game(3, S=13, max_depth=8, branch_lo=2, branch_hi=3, p_stop=0.15)


@pytest.mark.parametrize("game,early,late", [(gg.cfg1, 8, 40), (small, 150, 400)])
def test_a_solver_is_set_up_when_it_repays(cfr, game, early, late):
    s, ref = cfr.Solver(game()), cfr.Solver(game(), use_graph=False)
    for x in (s, ref):
        x.step(early, "cfr+", "alternating")
    assert s.resident_stats()["state"] == -1
    for x in (s, ref):
        x.step(late, "cfr+", "alternating")
    assert s.resident_stats()["state"] == 1
    assert s.get_state() == ref.get_state()
    s.close()
    ref.close()


def test_a_game_that_joins_is_charged_for(cfr):
    games = [gg.cfg1(), small(), gg.cfg1()]
    size = sum(cfr.Batch.game_size(g) for g in games)
    b = cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                  max_games=3, precision="fp64")
    first = b.add(games[0], "cfr+")
    b.run(4000)
    r = b.resident_stats(first)
    assert r["state"] == 1 and r["setups"] == 1
    late = b.add(games[1], "cfr+")
    b.run(100)
    r = b.resident_stats(late)
    assert r["setups"] == 1 and r["blocks"] == 0
    b.run(1000)
    r = b.resident_stats(late)
    assert r["state"] == 1 and r["setups"] == 2 and r["teams"] == 2
    # one that leaves costs nothing: the plans that are there go on
    b.remove(first)
    b.run(10)
    r = b.resident_stats(late)
    assert r["state"] == 1 and r["teams"] == 1 and r["setups"] == 2
    ref = cfr.Solver(games[1], use_graph=False)
    ref.step(1110, "cfr+", "alternating")
    for p in range(2):
        assert np.array_equal(b.strategy(late, p), ref.strategy(p, "average"))
    ref.close()
    b.close()
