"""The page-locked staging of downloads is allocated once, however the lengths
of the vectors come, and not for the first few of a small game."""
import numpy as np
import pytest

import gamegen as gg
from test_gpu_export import row

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


@pytest.mark.parametrize("n,first", [(3, 0), (32767, 0), (32768, 1), (65537, 1), (200000, 1)])
def test_one_allocation(cfr, n, first):
    game = row(n)  # two vectors: 3 sequences, and n
    s, ref = cfr.Solver(game), cfr.Solver(game, static_workspace=True)
    try:
        for k in range(4):
            for p in (0, 1):
                assert np.array_equal(s.strategy(p, "average"), ref.strategy(p, "average"))
            assert s.resident_stats()["stagings"] == (first if k == 0 else 1)
            for p in (0, 1):
                assert np.array_equal(s.regrets(p), ref.regrets(p))
            assert s.resident_stats()["stagings"] == 1
            for x in (s, ref):
                x.step(5, "cfr+", "alternating")
    finally:
        s.close()
        ref.close()


def test_one_allocation_in_a_batch(cfr):
    games = [row(n) for n in (10, 1000, 100, 40000, 70000)]
    size = sum(cfr.Batch.game_size(g) for g in games)
    b = cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                  max_games=len(games), precision="fp64")
    ids = [b.add(g, "cfr+") for g in games]
    b.run(20)
    for i, g in zip(ids, games):
        s = cfr.Solver(g)
        s.step(20, "cfr+", "alternating")
        for p in range(2):
            assert np.array_equal(b.strategy(i, p), s.strategy(p, "average"))
        s.close()
    assert b.resident_stats(ids[0])["stagings"] == 1
    b.close()
