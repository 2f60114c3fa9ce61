"""Chunks that give up waiting for the GPU (here: at once, for lack of any patience) are done by the kernel
that ends them, with the bits of the per-step launches and without a great loss of time: for T4 with one and
two elements per thread, H8, transversely isotropic materials, the thermal dose, several hundred patches,
and batches of which some scenarios have ended or end inside the chunk."""
import time

import numpy as np
import pytest

from paper_2009_10400_amd import workloads as W
from test_gpu_resident_paths import TI, problem, run

pytestmark = pytest.mark.gpu


def same(p, chunks, monkeypatch, **kw):
    want, _ = run(p, chunks, shared_update=2, **kw)
    monkeypatch.setenv("TLED_RESIDENT_WAIT_MS", "0")
    got, n = run(p, chunks, **kw)
    assert n == {"chunks": len(chunks), "given_up": len(chunks)}
    for k in want:
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("ti", [False, True])
@pytest.mark.parametrize("npe,patch,terms", [(4, 128, 1), (4, 504, 2), (4, 16, 4), (8, 0, 1), (8, 7, 3)])
def test_forms(npe, patch, terms, ti, monkeypatch):
    same(problem(npe, terms, ti), [4, 50, 7], monkeypatch, patch_elems=patch)


def test_dose(monkeypatch):
    same(W.spheres_t4(n=6), [50, 9], monkeypatch, dose=True)


def test_hundreds_of_patches(monkeypatch):
    p = W.ellipsoid_t4(50_000)
    p.params = dict(p.params, **TI)
    same(p, [50, 5], monkeypatch)


@pytest.mark.parametrize("graph_steps", [-1, 40])
def test_batch(graph_steps, monkeypatch):
    from paper_2009_10400_amd import tled
    sc = W.planning_scenarios(4, seed=5, lo=1500, hi=9000)
    out = []
    for wait in (None, "0"):
        if wait:
            monkeypatch.setenv("TLED_RESIDENT_WAIT_MS", wait)
        b = tled.Batch(0)
        b.set_options(graph_steps=graph_steps, shared_update=0 if wait else 2)
        for (p, _), n in zip(sc, [130, 61, 0, 205]):
            b.add(p, 2e-5, n)
        b.finalize()
        b.step(37)
        b.run()
        b.step(12)
        n = b.resident_counts()
        assert n["chunks"] == n["given_up"] and (n["chunks"] >= 4) == (wait is not None)
        out.append((b.read_all(), b.scenario_monitors(), b.monitors()))
        b.close()
    for (ua, Ta), (ub, Tb) in zip(out[0][0], out[1][0]):
        assert np.array_equal(ua, ub) and np.array_equal(Ta, Tb)
    assert all(np.array_equal(x, y) for x, y in zip(out[0][1], out[1][1]))
    for k in ("T_max", "T_min", "flags", "step"):
        assert out[0][2][k] == out[1][2][k], k
    for k in ("kinetic", "strain", "ablated_volume"):     # FP64 sums of the same terms in another order
        x, y = out[0][2][k], out[1][2][k]
        assert abs(x - y) <= 1e-12 * max(abs(x), 1e-300), k


def test_time_of_chunks_that_give_up(monkeypatch):
    """20 chunks of the 83k-tet ellipsoid: 9 ms with per-step launches, 4 s when one workgroup did the steps."""
    from paper_2009_10400_amd import tled
    monkeypatch.setenv("TLED_RESIDENT_WAIT_MS", "0")
    s = tled.from_problem(W.ellipsoid_t4(83_000), device=0)
    s.step(50)
    s.sync()
    t = time.perf_counter()
    s.step(1000)
    s.sync()
    t = time.perf_counter() - t
    print(f"  1000 steps in chunks that give up: {t * 1e3:.1f} ms")
    assert s.resident_counts() == {"chunks": 21, "given_up": 21}
    assert t < 0.5
    s.close()
