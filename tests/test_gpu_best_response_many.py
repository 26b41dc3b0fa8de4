"""Best responses of batches around the number of games whose levels one
launch looks through (1024 table entries of a player): a game's values are
those it has alone, bit for bit."""
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 340, 342, 511, 513, 1024, 1025, 2100])
def test_a_games_values_do_not_depend_on_how_many_there_are(n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    # two and three levels a player, one table entry each
    games = [gg.public_game(s, S=2, max_depth=4 + s % 3, branch_lo=2, branch_hi=2, p_stop=0.0)
             for s in range(3)]
    sizes = [cfr.Batch.game_size(g) for g in games]
    size = sum(sizes[i % 3] for i in range(n))
    b = cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                  max_games=n, precision="fp64", use_graph=False)
    ids = [b.add(games[i % 3], ("dcfr", "cfr+")[i % 2]) for i in range(n)]
    b.run(10)  # a check of all of them
    ref = {}
    for i, gid in enumerate(ids):
        kind = (i % 3, ("dcfr", "cfr+")[i % 2])
        if kind not in ref:
            s = cfr.Solver(games[kind[0]], use_graph=False)
            s.step(10, kind[1], "alternating")
            ref[kind] = s.exploitability("average")["expl"]
            s.close()
        assert b.status(gid)["expl"] == ref[kind], (n, i)
    b.close()
