"""A problem whose chunks could run in one kernel, on an allocator that has no memory for what only that
kernel needs (slots for the exchanged partials, their table, the meeting words, the temperature history of
the thermal dose): set up all the same, with the per-step launches' results and nothing held in vain."""
import numpy as np
import pytest

from paper_2009_10400_amd import workloads as W

pytestmark = pytest.mark.gpu


class Arena:
    """torch's allocator, up to a number of allocations."""

    def __init__(self, sim, limit=None):
        import torch
        from paper_2009_10400_amd import tled
        self.live, self.made = set(), 0

        def alloc(nbytes, ctx):
            if limit is not None and self.made >= limit:
                return None
            self.made += 1
            p = int(torch.cuda.caching_allocator_alloc(int(nbytes), 0))
            self.live.add(p)
            return p

        def free(p, ctx):
            self.live.remove(int(p))
            torch.cuda.caching_allocator_delete(int(p))

        self.cb = (tled._ALLOC(alloc), tled._FREE(free))
        assert tled._lib.tled_set_allocator(sim._h, self.cb[0], self.cb[1], None) == 0


def run(limit=None, extra=0, **options):
    import torch
    from paper_2009_10400_amd import tled
    torch.cuda.init()
    p = W.spheres_t4(n=6)
    s = tled.from_problem(p, device=0, finalize=False, **options)
    s.set_thermal_dose(7.39e39, 2.577e5)
    arena = Arena(s, None if limit is None else limit + extra)
    s.finalize()
    s.step(60)
    out = s.read_state()
    out["cem43"], out["omega"] = s.read_thermal_dose()
    held, made = s.info()["device_bytes"], arena.made
    live = len(arena.live)
    s.close()
    assert not arena.live
    return out, held, made, live


@pytest.mark.parametrize("extra", [0, 1, 2, 3])
def test_without_memory_for_the_resident_kernel(extra):
    want, held, made, live = run(shared_update=2)
    assert run()[2] == made + 4
    got, held2, made2, live2 = run(limit=made, extra=extra)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    assert made2 == made + extra and live2 == live and held2 == held
