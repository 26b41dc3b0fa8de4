"""Coded quads (8-bit codes into each block's values) against the plain quads:
a lone solver codes its stream where every block's values allow it, a batch
never does, and both take every sum in the same order, so the comparison is
exact."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


def matrix(kind):
    """2200 rows of 513 quads and 2051 of 550: over the coded form's smallest
    product, each row a long one for 8 nonzeros a thread and a block of its
    own for 16."""
    i, j = np.ogrid[:2200, :2051]
    rng = np.random.default_rng(3)
    # 255 values fill a block's codes, 256 are one too many (rows of the
    # matrix; its columns would have none to spare either way)
    M = {"255": 1.0 + (i + j) % 255, "256": 1.0 + (i + j) % 256,
         "holes": rng.integers(-3, 4, (2200, 2051)).astype(float),
         "signs": np.where(rng.random((2200, 2051)) < 0.5, 0.1, -0.1)}[kind]
    return gg.matrix_game(M)


def showdown():
    return gg.public_game(4, S=37, max_depth=7, branch_lo=3, branch_hi=4, p_stop=0.1,
                          payoff_kind="showdown")


GAMES = {"255": lambda: matrix("255"), "256": lambda: matrix("256"),
         "holes": lambda: matrix("holes"), "signs": lambda: matrix("signs"),
         "showdown": showdown}
# (stream bytes fall where the codes are used)
CODED = {"255": True, "256": False, "holes": True, "signs": True, "showdown": True}


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


@pytest.mark.parametrize("name", list(GAMES))
def test_coded_quads_equal_plain_quads(cfr, name):
    game = GAMES[name]()
    size = [int(v) for v in cfr.Batch.game_size(game)]
    for precision in ("fp64", "fp32", "fp32_acc64"):
        for items, perm in (([16, 8], [0, 1]), ([8, 16], [1, 0])):
            tiling = {"items": items, "rows": [256, 64], "vec": [3, 3], "perm": perm,
                      "xcd": [1, 0]}
            print(name, precision, items, flush=True)
            b = cfr.Batch(size[:2], size[2:4], size[4], max_games=1, precision=precision)
            b.tiling = tiling
            gid = b.add(game, "dcfr")
            b.run(7)
            s = cfr.Solver(game, precision=precision)
            s.tiling = tiling
            s.step(7, "dcfr", "alternating")
            assert s.exploitability("average") == b.exploitability(gid)
            for p in range(2):
                for k in ("current", "average"):
                    assert np.array_equal(s.strategy(p, k), b.strategy(gid, p, k))
            # eight bytes a quad and some for the values, or 20 (36)
            s.kernel_timing(True)
            b.kernel_timing(True)
            s.step(1, "dcfr", "alternating")
            b.run(1)
            for w in range(2):
                ratio = s.kernel_stats(w)[2] / b.kernel_stats(w)[2]
                assert ratio < 0.75 if CODED[name] else ratio == 1
            s.close()
            b.close()
