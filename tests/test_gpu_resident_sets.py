"""A batch whose games come, go and stop between runs, resident loop against a
launch per step: crowded first (teams that do not fit together are not used,
and nothing is held for them), then fewer games, then one."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


def large(seed):
    """62,000 sequences: a dozen of them need more than 256 workgroups, ten
    fit."""
    return gg.public_game(seed, S=24, max_depth=6, branch_lo=3, branch_hi=4, p_stop=0.0)


def units(seed):
    """196,000 sequences: four of them find no plan in a quarter of the chip."""
    return gg.public_game(seed, S=20, max_depth=8, branch_lo=3, branch_hi=3, p_stop=0.05)


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


class Pair:
    """The same calls on a batch that may use the loop and one that may not."""

    def __init__(self, cfr, games, precision):
        size = sum(cfr.Batch.game_size(g) for g in games)
        self.b = [cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                            max_games=len(games), precision=precision, use_graph=graph)
                  for graph in (True, False)]
        self.ids = []

    def add(self, game, variant="dcfr", **kw):
        got = [b.add(game, variant, **kw) for b in self.b]
        assert got[0] == got[1]
        self.ids.append(got[0])

    def remove(self, i):
        for b in self.b:
            b.remove(i)
        self.ids.remove(i)

    def run(self, n):
        for b in self.b:
            b.run(n)
        for i in self.ids:
            assert self.b[0].status(i) == self.b[1].status(i)
            for p in range(2):
                assert np.array_equal(self.b[0].strategy(i, p), self.b[1].strategy(i, p))

    def stats(self):
        assert self.b[1].resident_stats(self.ids[0])["launches"] == 0
        return self.b[0].resident_stats(self.ids[0])

    def close(self):
        for b in self.b:
            b.close()


def test_games_that_do_not_fit_together(cfr):
    games = [large(s) for s in range(12)]
    w = Pair(cfr, games, "fp32")
    for g in games:
        w.add(g, max_iterations=0)
    for _ in range(10):
        w.run(1000)
    r = w.stats()
    assert r["state"] == 0 and r["setups"] == 0 and r["device_bytes"] == 0
    # two leave: ten teams fit
    w.remove(w.ids[7])
    w.remove(w.ids[3])
    for _ in range(10):
        w.run(1000)
    r = w.stats()
    print(r, flush=True)
    assert r["state"] == 1 and r["teams"] == 10 and r["workgroups"] <= 256
    assert r["blocks"] > 1 and r["device_bytes"] > 0
    # they come back: nothing is held for teams that are not used
    w.add(games[3], variant="pcfr+")
    w.add(games[7], variant="cfr+", max_iterations=100)
    w.run(20)
    for _ in range(10):
        w.run(1000)
    r = w.stats()  # one of them stopped at 100
    assert r["state"] in (0, 1) and (r["state"] == 1 or r["teams"] == 0)
    # one is left: it gets all compute units
    few = r["blocks"]
    for i in w.ids[1:]:
        w.remove(i)
    for _ in range(10):
        w.run(1000)
    r = w.stats()
    print(r, few, flush=True)
    assert r["state"] == 1 and r["teams"] == 1 and r["blocks"] > max(few, 64)
    w.close()


def test_a_game_without_a_plan_in_its_share_gets_one_later(cfr):
    games = [units(s) for s in (10, 11, 12, 13)]
    w = Pair(cfr, games, "fp64")
    for g in games:
        w.add(g, "cfr+")
    for _ in range(4):
        w.run(1000)
    assert w.stats()["state"] == 0 and w.stats()["device_bytes"] == 0
    for i in w.ids[1:]:
        w.remove(i)
    for _ in range(2):
        w.run(1000)
    r = w.stats()
    print(r, flush=True)
    assert r["setups"] == 1
    assert r["blocks"] >= 128 if r["state"] == 1 else r["loop_ns"] > r["launches_ns"]
    w.close()


def test_a_game_whose_plan_costs_too_much_holds_nothing(cfr):
    """Its estimate is above the launches': the streams are not copied."""
    s = cfr.Solver(gg.public_game(6, S=40, max_depth=8, branch_lo=3, branch_hi=3, p_stop=0.0),
                   precision="fp32")
    for _ in range(3):
        s.step(1000, "cfr+", "alternating")
    r = s.resident_stats()
    assert r["state"] == 1 or (r["setups"] == 0 and r["device_bytes"] == 0)
    s.close()
