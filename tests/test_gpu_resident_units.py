"""Teams of the resident loop have to be on the chip all at once: on a stream
that may use a part of the compute units only, games that need a team launch
every step, and games of one workgroup still iterate inside one launch."""
import ctypes as C

import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("open_units", [None, 256, 255, 64])
def test_a_masked_stream(open_units):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    units = torch.cuda.get_device_properties(0).multi_processor_count
    handle = None
    if open_units is None:
        stream = torch.cuda.current_stream()
    else:
        hip = C.CDLL("libamdhip64.so")
        mask = (C.c_uint32 * 8)(*[(1 << max(0, min(32, open_units - 32 * w))) - 1 for w in range(8)])
        handle = C.c_void_p()
        if hip.hipExtStreamCreateWithCUMask(C.byref(handle), C.c_uint32(8), mask):
            pytest.skip("no stream with a mask")
        stream = torch.cuda.ExternalStream(handle.value)
    whole = open_units is None or open_units >= units
    for game, team in ((gg.cfg1(), False), (gg.cfg2_literal(), True)):
        s = cfr.Solver(game, stream=stream)
        ref = cfr.Solver(game, use_graph=False)
        s.step(2000, "pcfr+", "alternating")
        ref.step(2000, "pcfr+", "alternating")
        r = s.resident_stats()
        assert r["units"] == (min(units, 256) // 8 * 8 if whole else 1)
        assert r["state"] == (1 if whole or not team else 0)
        assert (r["blocks"] > 1) == (team and whole)
        for p in range(2):
            assert np.array_equal(s.strategy(p, "average"), ref.strategy(p, "average"))
        s.close()
        ref.close()
    if handle:
        torch.cuda.synchronize()
        assert hip.hipStreamDestroy(handle) == 0
