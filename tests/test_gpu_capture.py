"""Calls made while a stream is being captured into a graph: those that the
capture allowed before still leave it whole, and what they record replays with
the values that the host then holds."""
import ctypes

import pytest

from test_gpu_parity import Run, _task

pytestmark = pytest.mark.gpu

MODES = {"global": 0, "thread_local": 1, "relaxed": 2}


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_24532_amd as M
    M.lib()
    return M


class Capture:
    """A capture of `stream` (a new one if None) by the HIP runtime that the
    library is linked with."""

    def __init__(self, M, mode, stream=None):
        self.hip = ctypes.CDLL(M.LIB_PATH)
        self.stream, self.own = ctypes.c_void_p(stream), stream is None
        if self.own:
            assert self.hip.hipStreamCreateWithFlags(ctypes.byref(self.stream), 1) == 0
        assert self.hip.hipStreamBeginCapture(self.stream, MODES[mode]) == 0

    def end(self):
        """Status of the capture's end and the executable graph (None if broken)."""
        g, e = ctypes.c_void_p(), ctypes.c_void_p()
        rc = self.hip.hipStreamEndCapture(self.stream, ctypes.byref(g))
        if rc == 0 and g.value:
            assert self.hip.hipGraphInstantiate(ctypes.byref(e), g, None, None,
                                                ctypes.c_size_t(0)) == 0
            self.hip.hipGraphDestroy(g)
        else:
            self.hip.hipGetLastError()
        if self.own:
            self.hip.hipStreamDestroy(self.stream)
        return rc, e if e.value else None


@pytest.mark.parametrize("mode", sorted(MODES))
def test_contexts_come_and_go(M, mode):
    """Contexts created during another stream's capture, and bound ones (more
    than any that are kept for reuse) destroyed during it."""
    runs = [Run(M, [_task(2, 0, 2, 0.08, 0.0, k)], max_samples=1 << 12, max_iters=4)
            for k in range(5)]
    for r in runs:
        M.mbpt_integrate(r.set, 1 << 12, 1)
    print(f"case contexts mode={mode}", flush=True)
    cap = Capture(M, mode)
    ctx = M.mbpt_context_create()
    M.mbpt_context_destroy(ctx)
    for r in runs:
        r.close()
    assert cap.end()[0] == 0
    # and the blocks that were kept serve the next contexts
    again = [Run(M, [_task(2, 0, 2, 0.08, 0.0, k)], max_samples=1 << 12, max_iters=4)
             for k in range(3)]
    for k, r in enumerate(again):
        per, _ = M.mbpt_integrate(r.set, 1 << 12, 1)
        assert per[0].iters_done == 1 and per[0].n_evals == 1 << 12
    for r in again:
        r.close()


def test_training_set_in_a_capture(M):
    """mbpt_set_training does not wait for the stream, so it may be captured: the
    graph's replays upload the parameters that the host holds at the time, and a
    run with replays between its calls (which use the staging of their own copies)
    gives what the run without them gives."""
    N = 1 << 13

    def run(replays):
        r = Run(M, [_task(2, 0, 2, 0.08, 0.0, k) for k in range(3)], max_samples=N, max_iters=16)
        out = []
        try:
            M.mbpt_integrate(r.set, N, 1)
            if replays:
                cap = Capture(M, "thread_local", r.stream.cuda_stream)
                M.mbpt_set_training(r.set, 3)
                rc, graph = cap.end()
                assert rc == 0 and graph is not None
            else:
                M.mbpt_set_training(r.set, 3)
            for k in range(4):
                if k == 2:
                    M.mbpt_set_density(r.set, 0.1)
                if replays:
                    assert cap.hip.hipGraphLaunch(graph, cap.stream) == 0
                per, _ = M.mbpt_integrate(r.set, N, 2)
                out.append([(p.iters_done, p.n_evals, p.E_per_A, p.sigma) for p in per])
            if replays:
                r.stream.synchronize()
                cap.hip.hipGraphExecDestroy(graph)
        finally:
            r.close()
        return out

    want, got = run(False), run(True)
    for a, b in zip(want, got):
        for x, y in zip(a, b):
            assert x[:2] == y[:2]
            assert y[2:] == pytest.approx(x[2:], rel=1e-9)
