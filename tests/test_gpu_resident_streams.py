"""Solvers and a batch whose teams take most of the chip, on streams and
threads of their own at once: each iterates as it does alone."""
import threading

import numpy as np
import pytest

import gamegen as gg
from test_gpu_resident import GAMES

pytestmark = pytest.mark.gpu


def test_teams_on_several_streams():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    games = {"units": (GAMES["units"](), 900), "long-rows": (GAMES["long-rows"](), 2000),
             "d8": (gg.cfg2_literal(), 4000), "tiny": (gg.cfg1(), 6000)}
    want = {}
    for name, (game, n) in games.items():
        s = cfr.Solver(game, use_graph=False)
        s.step(n, "cfr+", "alternating")
        want[name] = [s.strategy(p, "average") for p in range(2)]
        s.close()
    got, teams, errors = {}, {}, []

    def solve(key, name):
        try:
            game, n = games[name]
            stream = torch.cuda.Stream()
            s = cfr.Solver(game, stream=stream)
            done = 0
            while done < n:
                k = min(n - done, 700 if done == 0 else 50)
                s.step(k, "cfr+", "alternating")
                done += k
            got[key] = [s.strategy(p, "average") for p in range(2)]
            teams[key] = s.resident_stats()["blocks"]
            s.close()
        except Exception as e:  # reported below
            errors.append((key, e))

    threads = [threading.Thread(target=solve, args=((name, i), name))
               for name in games for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not any(t.is_alive() for t in threads) and not errors
    assert sum(b > 1 for b in teams.values()) >= 4
    for (name, i), v in got.items():
        for p in range(2):
            assert np.array_equal(v[p], want[name][p]), (name, i, p)


def test_streams_that_come_and_go():
    """One stream with two solvers, then a second and a third stream, without
    waits between their calls."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    game, n = GAMES["units"](), 900
    ref = cfr.Solver(game, use_graph=False)
    want = {}
    for done in (n, n + 50, n + 100):
        ref.step(done - ref.iteration, "cfr+", "alternating")
        want[done] = [ref.strategy(p, "average") for p in range(2)]
    ref.close()
    streams = [torch.cuda.Stream() for _ in range(3)]

    def check(s, done):
        assert s.resident_stats()["blocks"] > 1
        for p in range(2):
            assert np.array_equal(s.strategy(p, "average"), want[done][p])

    a, b = (cfr.Solver(game, stream=streams[0]) for _ in range(2))
    for s in (a, b):
        s.step(n, "cfr+", "alternating")
    c = cfr.Solver(game, stream=streams[1])
    c.step(n, "cfr+", "alternating")
    for s in (a, c, b, c, a):  # c 100 more, a 100, b 50
        s.step(50, "cfr+", "alternating")
    check(a, n + 100)
    check(b, n + 50)
    check(c, n + 100)
    a.close()
    b.close()
    d = cfr.Solver(game, stream=streams[2])
    for s, k in ((c, 0), (d, n), (d, 50)):
        s.step(k, "cfr+", "alternating")
    check(d, n + 50)
    c.close()
    d.step(50, "cfr+", "alternating")
    check(d, n + 100)
    d.close()
