"""Several handles of one process on streams of their own: chunks in the resident kernel run side by side where
they fit, take the per-step launches where they do not, and none gives up; the results are those of the
handles alone.  A handle leaves the streams of the others alone."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2009_10400_amd import workloads as W

pytestmark = pytest.mark.gpu


def small():
    return W.cube_t4(n=7)


def large():
    return W.ellipsoid_t4(83_000)          # about 650 patches of the thousand that are resident at once


def alone(p, steps):
    from paper_2009_10400_amd import tled
    s = tled.from_problem(p, device=0, shared_update=2)
    s.step(steps)
    out = s.read_state()
    s.close()
    return out


def handles(p, n):
    import torch
    from paper_2009_10400_amd import tled
    streams = [torch.cuda.Stream() for _ in range(n)]
    return streams, [tled.from_problem(p, device=0, stream=st.cuda_stream) for st in streams]


@pytest.mark.parametrize("n", [2, 4, 7])
def test_small_problems_all_run_resident(n):
    p = small()
    want = alone(p, 300)
    streams, sims = handles(p, n)
    for _ in range(6):
        for s in sims:
            s.step(50)
    for s in sims:
        got = s.read_state()
        assert all(np.array_equal(got[k], want[k]) for k in want)
        assert s.resident_counts() == {"chunks": 6, "given_up": 0}
    for s in sims:
        s.close()


@pytest.mark.parametrize("n", [2, 3, 5])
def test_large_problems_do_not_wait_for_each_other(n):
    p = large()
    want = alone(p, 300)
    streams, sims = handles(p, n)
    for _ in range(6):
        for s in sims:
            s.step(50)
    counts = []
    for s in sims:
        got = s.read_state()
        assert all(np.array_equal(got[k], want[k]) for k in want)
        counts.append(s.resident_counts())
    assert all(c["given_up"] == 0 for c in counts)
    assert sum(c["chunks"] for c in counts) < 6 * n         # not all of them at once
    for s in sims[1:]:
        s.close()
    before = counts[0]["chunks"]
    sims[0].step(100)                                       # alone again
    sims[0].sync()
    assert sims[0].resident_counts() == {"chunks": before + 2, "given_up": 0}
    sims[0].close()


def test_handles_on_one_stream_all_run_resident():
    import torch
    from paper_2009_10400_amd import tled
    p = large()
    want = alone(p, 150)
    st = torch.cuda.Stream()
    sims = [tled.from_problem(p, device=0, stream=st.cuda_stream) for _ in range(2)]
    for _ in range(3):
        for s in sims:
            s.step(50)
    for s in sims:
        got = s.read_state()
        assert all(np.array_equal(got[k], want[k]) for k in want)
        assert s.resident_counts() == {"chunks": 3, "given_up": 0}
        s.close()


def test_threads_with_a_handle_each():
    p = small()
    want = alone(p, 500)
    streams, sims = handles(p, 4)
    got = [None] * 4

    def work(i):
        for n in (50, 130, 4, 16, 300):
            sims[i].step(n)
        got[i] = sims[i].read_state()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g, s in zip(got, sims):
        assert all(np.array_equal(g[k], want[k]) for k in want)
        assert s.resident_counts()["given_up"] == 0
        s.close()


def test_another_handles_stream_under_capture():
    """A handle is set up and run while the owner of the only other one's stream captures it."""
    from paper_2009_10400_amd import tled
    hip = ctypes.CDLL(None)                 # the process's own HIP runtime, loaded with the library
    p = small()
    want = alone(p, 100)
    (st,), (a,) = handles(p, 1)
    a.step(50)
    a.sync()
    a.step(50)
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(st.cuda_stream), 2) == 0      # hipStreamCaptureModeRelaxed
    b = tled.from_problem(p, device=0)
    b.step(100)
    got = b.read_state()
    graph, nodes = ctypes.c_void_p(), ctypes.c_size_t(7)
    assert hip.hipStreamEndCapture(ctypes.c_void_p(st.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert nodes.value == 0                 # nothing of b's in the owner's graph
    assert hip.hipGraphDestroy(graph) == 0
    for s in (a, b):
        assert s.resident_counts() == {"chunks": 2, "given_up": 0}
        out = s.read_state()
        assert all(np.array_equal(out[k], want[k]) for k in want)
    assert all(np.array_equal(got[k], want[k]) for k in want)
    a.close()
    b.close()
