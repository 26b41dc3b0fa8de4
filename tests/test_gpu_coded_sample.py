"""Coded quads are sought in a sample of the blocks first: one block with too
many values keeps its product's plain quads, whether the sample holds it or
not, and the other product is coded."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row", [None, 0, 1, 1001, 2199])
@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64"])
def test_one_block_with_too_many_values(precision, row):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    M = np.random.default_rng(3).integers(-3, 4, (2200, 2051)).astype(float)
    if row is not None:
        M[row] = 10.0 + np.arange(2051) % 300
    game = gg.matrix_game(M)
    size = [int(v) for v in cfr.Batch.game_size(game)]
    tiling = {"items": [16, 16], "rows": [256, 256], "vec": [3, 3], "perm": [0, 1], "xcd": [1, 1]}
    b = cfr.Batch(size[:2], size[2:4], size[4], max_games=1, precision=precision)
    b.tiling = tiling
    gid = b.add(game, "cfr+")
    b.run(5)
    s = cfr.Solver(game, precision=precision)
    s.tiling = tiling
    s.step(5, "cfr+", "alternating")
    for p in range(2):
        for k in ("current", "average"):
            assert np.array_equal(s.strategy(p, k), b.strategy(gid, p, k))
    assert s.exploitability("average") == b.exploitability(gid)
    s.kernel_timing(True)
    b.kernel_timing(True)
    s.step(1, "cfr+", "alternating")
    b.run(1)
    ratio = [s.kernel_stats(w)[2] / b.kernel_stats(w)[2] for w in range(2)]
    assert ratio[0] == 1 if row is not None else ratio[0] < 0.75
    assert ratio[1] < 0.75
    s.close()
    b.close()
