"""Iterations asked for while the caller captures the solver's stream: nothing
is set up for the resident loop then (that allocates and waits, which ends a
capture).  A solver that launches every step is recorded and replayed; one
with a graph of its own (whose launches the runtime does not record) goes on
the same afterwards, and takes the loop."""
import ctypes as C

import numpy as np
import pytest

import gamegen as gg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("set_up_before", [False, True])
def test_a_captured_step(use_graph, set_up_before):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_14277_amd as cfr
    hip = C.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    st = C.c_void_p(stream.cuda_stream)
    s = cfr.Solver(gg.cfg1(), stream=stream, use_graph=use_graph)
    ref = cfr.Solver(gg.cfg1(), use_graph=False)
    done = 3
    s.step(3, "cfr+", "alternating")
    if set_up_before:
        s.step(1000, "cfr+", "alternating")
        done += 1000
    torch.cuda.synchronize()
    before = s.resident_stats()
    assert before["state"] == (-1 if not set_up_before else 1 if use_graph else 0)
    graph, ex = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamBeginCapture(st, 1) == 0  # thread-local
    try:
        s.step(1000, "cfr+", "alternating")
        during = s.resident_stats()
    finally:
        rc = hip.hipStreamEndCapture(st, C.byref(graph))
    assert rc == 0 and during == before
    if not use_graph:
        assert hip.hipGraphInstantiate(C.byref(ex), graph, None, None, C.c_size_t(0)) == 0
        for _ in range(3):
            assert hip.hipGraphLaunch(ex, st) == 0
            torch.cuda.synchronize()
            done += 1000
        assert hip.hipGraphExecDestroy(ex) == 0
        ref.step(done, "cfr+", "alternating")
    else:
        torch.cuda.synchronize()
        ref.set_state(s.get_state())
    assert hip.hipGraphDestroy(graph) == 0
    for n in (0, 1000):
        if n:
            s.step(n, "cfr+", "alternating")
            ref.step(n, "cfr+", "alternating")
        for p in range(2):
            for kind in ("current", "average"):
                assert np.array_equal(s.strategy(p, kind), ref.strategy(p, kind))
    assert s.resident_stats()["launches"] == before["launches"] + (1 if use_graph else 0)
    s.close()
    ref.close()
