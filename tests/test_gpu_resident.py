"""Chunks of steps in one kernel (problems whose patches are all resident on the GPU at once) against
the same chunks with one patch and one shared-node launch per step: the same bits, for both element
types, one and two elements per thread, partial patches, every chunk length around the shortest one
taken, the thermal dose, several streams, and batches whose scenarios end inside a chunk.

shared_update=2 asks for a shared-node kernel after every step and so keeps the per-step launches."""
import numpy as np
import pytest

from paper_2009_10400_amd import workloads as W

pytestmark = pytest.mark.gpu


def problem(name):
    p = {
        "t4_one_patch_edge": lambda: W.cube_t4(n=3),            # 162 elements: a full and a partial patch of 128
        "t4_cube": lambda: W.cube_t4(n=7),                      # 2058 elements, one Prony term
        "t4_ellipsoid": lambda: W.ellipsoid_t4(20000),          # irregular, two Prony terms, shrinkage
        "t4_no_prony": lambda: W.cube_t4(n=6),
        "t4_ti": lambda: W.cube_t4(n=6),
        "h8_cube": lambda: W.cube_h8(n=9),                      # 729 elements: partial patch
        "h8_ti": lambda: W.cube_h8(n=8),
    }[name]()
    if name == "t4_ellipsoid":
        p.params = dict(p.params, shrink_T=p.params["T0"] + 0.05, shrink_width=0.5)
    if name == "t4_no_prony":
        p.params = dict(p.params, g=[], tau=[], n_prony=0)
    if name.endswith("_ti"):
        p.params = dict(p.params, expan_mode=1, alpha_m=3e-4, cond_mode=1, k_m=1.5)
    return p


def fields(p, chunks, dose=False, state=None, **options):
    from paper_2009_10400_amd import tled
    s = tled.from_problem(p, device=0, finalize=False, **options)
    if dose:
        s.set_thermal_dose(7.39e39, 2.577e5)
    s.finalize()
    if state:
        u, up, T = W.random_state(p, 3, 2e-5, 30.0)
        s.write_state(u=u, v=(u - up) / s.dt * 1e-3, T=T)
    for n in chunks:
        s.step(n)
    out = s.read_state()
    mon = s.monitors()
    if dose:
        out["cem43"], out["omega"] = s.read_thermal_dose()
    s.close()
    return out, mon


def same(a, b):
    (x, mx), (y, my) = a, b
    for k in x:
        assert np.array_equal(x[k], y[k]), (k, np.abs(np.asarray(x[k]) - y[k]).max())
    assert mx["step"] == my["step"] and mx["flags"] == my["flags"]
    assert mx["T_max"] == my["T_max"] and mx["T_min"] == my["T_min"]
    for k in ("kinetic", "strain", "ablated_volume"):     # FP64 sums of the same terms in another order
        assert abs(mx[k] - my[k]) <= 1e-12 * max(abs(mx[k]), 1e-300), (k, mx[k], my[k])


@pytest.mark.parametrize("patch", [0, 200, 256, 264, 504])
@pytest.mark.parametrize("name", ["t4_one_patch_edge", "t4_cube", "t4_ellipsoid", "t4_no_prony", "t4_ti"])
def test_t4_same_bits(name, patch):
    p = problem(name)
    runs = [fields(p, [3, 4, 5, 50, 61], state=True, patch_elems=patch, shared_update=su) for su in (0, 2)]
    assert np.abs(runs[0][0]["u"]).max() > 1e-6
    same(*runs)


@pytest.mark.parametrize("patch", [0, 60, 128])
@pytest.mark.parametrize("name", ["h8_cube", "h8_ti"])
def test_h8_same_bits(name, patch):
    p = problem(name)
    same(*(fields(p, [4, 7, 50, 22], state=True, patch_elems=patch, shared_update=su) for su in (0, 2)))


def test_dose_same_bits():
    p = W.spheres_t4(n=6)
    same(*(fields(p, [50, 9, 3], dose=True, state=True, shared_update=su) for su in (0, 2)))


def test_chunks_that_give_up_waiting_are_done_all_the_same(monkeypatch):
    """With no patience every chunk gives up before its first step (until a read tells the host), and
    the kernel that ends the chunk does the steps."""
    p = problem("t4_cube")
    want = fields(p, [6, 10], dose=True, state=True, shared_update=2)
    monkeypatch.setenv("TLED_RESIDENT_WAIT_MS", "0")
    same(fields(p, [6, 10], dose=True, state=True), want)


def test_two_problems_in_turn_on_their_own_streams():
    from paper_2009_10400_amd import tled
    p, q = problem("t4_ellipsoid"), problem("h8_cube")
    want = [fields(x, [50] * 6, shared_update=2)[0] for x in (p, q)]
    sims = [tled.from_problem(x, device=0) for x in (p, q)]
    for _ in range(6):
        for s in sims:
            s.step(50)
    for s, w in zip(sims, want):
        assert np.array_equal(s.read_u(), w["u"]) and np.array_equal(s.read_T(), w["T"])
    sims[0].close()
    sims[1].step(50)
    sims[1].sync()


def test_rewound_state_does_not_meet_old_partials():
    """A slot of the exchange is empty until its partial of the step is written, and a chunk empties all
    slots before its first step; going back to an earlier state must not find partials of the first
    pass over the same steps."""
    from paper_2009_10400_amd import tled
    p = problem("t4_cube")
    s = tled.from_problem(p, device=0)
    s.step(10)
    blob = s.get_state()
    s.step(50)
    first = s.read_state()
    s.set_state(blob)
    u, up, T = W.random_state(p, 5, 1e-5, 5.0)
    s.write_state(u=u, T=T, step=10)
    s.step(50)
    s.set_state(blob)
    s.step(50)
    again = s.read_state()
    for k in first:
        assert np.array_equal(first[k], again[k]), k


@pytest.mark.parametrize("graph_steps", [-1, 40])
def test_batch_same_bits(graph_steps):
    from paper_2009_10400_amd import tled
    sc = W.planning_scenarios(4, seed=5, lo=1500, hi=9000)
    out = []
    for su in (0, 2):
        b = tled.Batch(0)
        b.set_options(graph_steps=graph_steps, shared_update=su)
        for (p, _), n in zip(sc, [130, 61, 0, 205]):
            b.add(p, 2e-5, n)
        b.finalize()
        b.step(37)
        b.run()
        b.step(12)
        out.append((b.read_all(), b.scenario_monitors()))
        b.close()
    for (ua, Ta), (ub, Tb) in zip(out[0][0], out[1][0]):
        assert np.array_equal(ua, ub) and np.array_equal(Ta, Tb)
    assert all(np.array_equal(x, y) for x, y in zip(out[0][1], out[1][1]))
