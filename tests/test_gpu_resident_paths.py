"""Which way chunks of steps run, as counted by the library, for every form of the resident kernel, so that
the comparisons of it with the per-step launches compare two ways: T4 with one and two elements per thread,
H8, transversely isotropic expansion and conduction, no to four Prony terms, the thermal dose, batches."""
import numpy as np
import pytest

from paper_2009_10400_amd import workloads as W

pytestmark = pytest.mark.gpu

NO_TERMS = dict(g=[], tau=[], n_prony=0)
TERMS = {0: NO_TERMS, 1: dict(g=[0.5], tau=[0.58], n_prony=1), 2: dict(g=[0.3, 0.2], tau=[0.58, 2.0], n_prony=2),
         3: dict(g=[0.3, 0.2, 0.1], tau=[0.58, 2.0, 7.0], n_prony=3),
         4: dict(g=[0.3, 0.2, 0.1, 0.1], tau=[0.58, 2.0, 7.0, 20.0], n_prony=4)}
TI = dict(expan_mode=1, alpha_m=3e-4, cond_mode=1, k_m=1.5)


def problem(npe, terms, ti=False):
    p = W.cube_t4(n=7) if npe == 4 else W.cube_h8(n=9)
    p.params = dict(p.params, **TERMS[terms], **(TI if ti else {}))
    return p


def run(p, chunks, dose=False, **options):
    from paper_2009_10400_amd import tled
    s = tled.from_problem(p, device=0, finalize=False, **options)
    if dose:
        s.set_thermal_dose(7.39e39, 2.577e5)
    s.finalize()
    u, up, T = W.random_state(p, 3, 2e-5, 30.0)
    s.write_state(u=u, v=(u - up) / s.dt * 1e-3, T=T)
    for n in chunks:
        s.step(n)
    out = s.read_state()
    if dose:
        out["cem43"], out["omega"] = s.read_thermal_dose()
    counts = s.resident_counts()
    s.close()
    return out, counts


# steps of 3 (too short), 4, 50, and 61 in chunks of 50 and 11
CHUNKS, RESIDENT = [3, 4, 50, 61], 4


@pytest.mark.parametrize("terms", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("ti", [False, True])
@pytest.mark.parametrize("npe,patch", [(4, 128), (4, 504), (8, 0)])
def test_every_form_runs_and_gives_the_same_bits(npe, patch, ti, terms):
    p = problem(npe, terms, ti)
    got, n = run(p, CHUNKS, patch_elems=patch)
    want, none = run(p, CHUNKS, patch_elems=patch, shared_update=2)
    two = npe == 4 and patch > 256                 # two elements per thread: state of at most two terms in registers
    assert n == {"chunks": 0 if two and terms > 2 else RESIDENT, "given_up": 0}
    assert none == {"chunks": 0, "given_up": 0}
    assert np.abs(got["u"]).max() > 1e-6
    for k in want:
        assert np.array_equal(got[k], want[k]), k


def test_dose_and_batch_run():
    from paper_2009_10400_amd import tled
    assert run(W.spheres_t4(n=6), CHUNKS, dose=True)[1] == {"chunks": RESIDENT, "given_up": 0}
    for graph_steps, n in ((-1, 3), (40, 4)):      # 37 steps, then 93 in chunks of 100 or 40
        b = tled.Batch(0)
        b.set_options(graph_steps=graph_steps)
        for p, _ in W.planning_scenarios(3, seed=5, lo=1500, hi=9000):
            b.add(p, 2e-5, 130)
        b.finalize()
        b.step(37)
        b.run()
        b.step(12)
        assert b.resident_counts() == {"chunks": n + (graph_steps > 0), "given_up": 0}
        b.close()


def test_no_patience_gives_every_chunk_up(monkeypatch):
    p = problem(4, 1)
    want, _ = run(p, [60], shared_update=2)
    monkeypatch.setenv("TLED_RESIDENT_WAIT_MS", "0")
    got, n = run(p, [60])
    assert n == {"chunks": 2, "given_up": 2}
    for k in want:
        assert np.array_equal(got[k], want[k]), k


@pytest.mark.parametrize("steps", [4, 5, 6, 49])
def test_slots_of_an_earlier_chunk_are_not_met(steps):
    """A chunk empties its slots before its workgroups meet, whatever the one before left in the three buffers
    (its length modulo 3 decides which it used last)."""
    from paper_2009_10400_amd import tled
    p = problem(4, 1)
    want = None
    for su in (2, 0):
        s = tled.from_problem(p, device=0, shared_update=su)
        s.step(10)
        blob = s.get_state()
        out = []
        for n in (steps, steps + 1, steps):
            s.set_state(blob)
            u, _, T = W.random_state(p, 5 + n, 1e-5, 5.0)
            s.write_state(u=u, T=T, step=10)
            s.step(n)
            out.append(s.read_state())
        s.close()
        if want:
            for a, b in zip(out, want):
                assert all(np.array_equal(a[k], b[k]) for k in a)
        want = out
