"""Sequential sums over coded quads at every row length: rows of 1 to 513 quads
(whole batches of reads, remainders, long rows), few and many to a block, equal
the plain quads exactly."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,order", [("fp64", "default"), ("fp32", "sequential"),
                                             ("fp32_acc64", "sequential")])
@pytest.mark.parametrize("lengths", ["all", "short", "mixed"])
def test_rows_of_every_length(precision, order, lengths):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    rng = np.random.default_rng(11)
    rows, cols = (2200, 2051) if lengths == "all" else (24000, 140)
    M = rng.integers(1, 8, (rows, cols)).astype(float) * rng.choice([-1.0, 1.0], (rows, cols))
    n = {"all": 1 + np.arange(rows) % cols, "short": np.full(rows, cols),
         "mixed": np.where(np.arange(rows) % 70 < 3, cols, 1 + np.arange(rows) % cols)}[lengths]
    M[np.arange(cols)[None, :] >= n[:, None]] = 0.0
    game = gg.matrix_game(M)
    size = [int(v) for v in cfr.Batch.game_size(game)]
    for items in ([16, 8], [8, 16]):
        tiling = {"items": items, "rows": [256, 64], "vec": [3, 3], "perm": [1, 1], "xcd": [0, 1]}
        b = cfr.Batch(size[:2], size[2:4], size[4], max_games=1, precision=precision,
                      spmv_order=order)
        b.tiling = tiling
        gid = b.add(game, "pcfr+")
        b.run(5)
        s = cfr.Solver(game, precision=precision, spmv_order=order)
        s.tiling = tiling
        s.step(5, "pcfr+", "alternating")
        for p in range(2):
            for k in ("current", "average"):
                assert np.array_equal(s.strategy(p, k), b.strategy(gid, p, k))
        assert s.exploitability("average") == b.exploitability(gid)
        s.kernel_timing(True)
        b.kernel_timing(True)
        s.step(1, "pcfr+", "alternating")
        b.run(1)
        assert all(s.kernel_stats(w)[2] < 0.8 * b.kernel_stats(w)[2] for w in range(2))
        s.close()
        b.close()
