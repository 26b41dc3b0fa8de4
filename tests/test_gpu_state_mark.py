"""The word of a game's scalars in which a failed team of the resident loop
leaves its mark belongs to the device: a saved state brings none with it."""
import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu

# the image: a header of 72 bytes, then the scalars: eight doubles, the
# variant, the averaging kind, and the two words in question
PAD = slice(72 + 8 * 8 + 2 * 4, 72 + 8 * 8 + 4 * 4)


@pytest.mark.parametrize("word", [b"\1\0\0\0\0\0\0\0", b"\377" * 8])
def test_an_images_padding_is_not_read_as_a_failure(word):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    a, b = (cfr.Solver(gg.cfg1()) for _ in range(2))
    a.step(200, "dcfr", "alternating")
    image = a.get_state()
    assert image[PAD] == bytes(8)
    b.set_state(image[:PAD.start] + word + image[PAD.stop:])
    for s in (a, b):
        s.step(200, "dcfr", "alternating")
    assert a.exploitability("average") == b.exploitability("average")
    for p in range(2):
        assert np.array_equal(a.strategy(p, "average"), b.strategy(p, "average"))
    assert a.get_state() == b.get_state()
    a.close()
    b.close()
