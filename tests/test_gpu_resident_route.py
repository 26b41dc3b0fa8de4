"""Which way the iterations of a solver or a batch run, and that results do
not depend on it: the games of test_gpu_resident.py take the structures that
they are there for, and the state is that of a launch per step."""
import numpy as np
import pytest

import gamegen as gg
from test_gpu_resident import GAMES, QUADS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


# workgroups of the team, from and to
TEAMS = {"tiny": (1, 1), "matrix": (1, 1), "one-group": (2, 32), "d8": (2, 32), "deep": (2, 32),
         "wide": (2, 32), "actions-64": (1, 1), "actions-65": (0, 0), "long-rows": (64, 256),
         "showdown": (2, 32), "depth-first": (2, 32), "units": (64, 256)}


@pytest.mark.parametrize("name", list(GAMES))
def test_the_structure_meant_for_each_game_runs(cfr, name):
    lo, hi = TEAMS[name]
    s = cfr.Solver(GAMES[name]())
    for _ in range(4):
        s.step(1000, "cfr+", "alternating")
    s.exploitability()
    r = s.resident_stats()
    print(name, r, flush=True)
    assert r["state"] == (1 if hi else 0)
    assert lo <= r["blocks"] <= hi
    assert (r["launches"] > 0) == bool(hi)
    if name in ("deep", "units"):
        assert r["cut0"] + r["cut1"] > 0
    s.close()


def test_quads_are_read_where_the_tiling_has_them(cfr):
    s = cfr.Solver(GAMES["showdown"](), precision="fp32_acc64")
    s.tiling = QUADS
    s.step(3000, "dcfr", "alternating")
    r = s.resident_stats()
    assert (r["state"], r["quads0"], r["quads1"]) == (1, 1, 1)
    s.close()


@pytest.mark.parametrize("n,launches", [(1024, 1), (1025, 2), (2500, 3)])
def test_a_long_step_is_split(cfr, n, launches):
    a = cfr.Solver(gg.cfg1())
    b = cfr.Solver(gg.cfg1(), use_graph=False)
    a.step(100, "cfr+", "alternating")  # set up here
    before = a.resident_stats()
    assert before["state"] == 1
    a.step(n, "cfr+", "alternating")
    assert a.resident_stats()["launches"] - before["launches"] == launches
    b.step(100 + n, "cfr+", "alternating")
    assert a.get_state() == b.get_state()
    assert b.resident_stats()["launches"] == 0
    a.close()
    b.close()


def test_options_that_keep_a_launch_per_step(cfr):
    for kw in ({"use_graph": False}, {"down_pass": "levels"}, {"up_pass": "levels"},
               {"static_workspace": True}):
        s = cfr.Solver(gg.cfg1(), **kw)
        s.step(3000, "cfr+", "alternating")
        assert s.resident_stats()["launches"] == 0, kw
        s.close()
