"""Downloads of strategies and regrets (converted on the device into page-
locked memory, in parts) against a static solver, which allocates nothing and
copies plainly: the same doubles."""
import numpy as np
import pytest

import gamegen as gg
from helpers import dfs_renumber

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfr():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as m
    return m


def row(n):
    """2 x (n - 1) actions: n sequences for the second player."""
    return gg.matrix_game(np.random.default_rng(n).normal(size=(2, n - 1)))


# a part is 65536 sequences; two are in flight
GAMES = {"one": lambda: row(65535), "full": lambda: row(65536), "full+1": lambda: row(65537),
         "two+1": lambda: row(131073), "three+1": lambda: row(196609), "tiny": gg.cfg1,
         "permuted": lambda: dfs_renumber(gg.public_game(5, S=40, max_depth=8, branch_lo=2,
                                                         branch_hi=3, p_stop=0.1)),
         }


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32_acc64"])
@pytest.mark.parametrize("name", list(GAMES))
def test_downloads_equal_plain_copies(cfr, name, precision):
    game = GAMES[name]()
    a = cfr.Solver(game, precision=precision)
    b = cfr.Solver(game, precision=precision, static_workspace=True)
    try:
        for n in (0, 1, 4):
            if n:
                a.step(n, "cfr+", "alternating")
                b.step(n, "cfr+", "alternating")
            for p in (1, 0):  # the larger one first, then one that fits its staging
                for kind in ("current", "average"):
                    assert np.array_equal(a.strategy(p, kind), b.strategy(p, kind)), (n, p, kind)
                assert np.array_equal(a.regrets(p), b.regrets(p)), (n, p)
    finally:
        a.close()
        b.close()
