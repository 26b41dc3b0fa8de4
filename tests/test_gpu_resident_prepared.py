"""A prepared game may be added any number of times: each copy iterates in the
resident loop from plans of its own, and equals the game added directly."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_acc64"])
def test_added_twice_and_directly(precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    from paper_2605_14277_amd import serve
    game = gg.public_game(6, S=5, max_depth=6, branch_lo=2, branch_hi=3, p_stop=0.2)
    size = 3 * cfr.Batch.game_size(game)
    b = cfr.Batch([int(v) for v in size[:2]], [int(v) for v in size[2:4]], int(size[4]),
                  max_games=3, precision=precision)
    p = serve.Prepared(game, precision)
    ids = [serve.add_prepared(b, p, "dcfr") for _ in range(2)]
    p.close()
    direct = b.add(game, "dcfr")
    b.run(3000)
    ref = cfr.Solver(game, precision=precision, use_graph=False)
    ref.step(3000, "dcfr", "alternating")
    for i in (*ids, direct):
        r = b.resident_stats(i)
        assert r["state"] == 1 and r["teams"] == 3 and r["blocks"] >= 1
        for q in range(2):
            assert np.array_equal(b.strategy(i, q), ref.strategy(q, "average"))
    ref.close()
    b.close()
