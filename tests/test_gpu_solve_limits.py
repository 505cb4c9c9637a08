"""Solves at the limits of what their entry points accept: the largest
iteration cap."""
import pytest

import paper_1810_05370_amd as tm
import synthetic
from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


def _sim(n, precision, P=None, **kw):
    """A context with a tumour and an elasticity force, at rest."""
    return tm.from_inputs(synthetic.workload_inputs("seeds3_n128", n=n), P or synthetic.params(), precision=precision, **kw)


@pytest.mark.parametrize("n", [16, 128])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_the_largest_iteration_cap_is_a_cap_that_is_never_met(n, precision):
    """max_it = 2^31 - 1 gives the bits of max_it = 1000, in the elasticity solve and in split steps."""
    torch = need_gpu()
    got = []
    for cap in (1000, 2 ** 31 - 1):
        say(f"cap {cap}, n={n}, {precision}")
        sim = _sim(n, precision, max_it=cap)
        u, it, rr = sim.solve_elasticity()
        st = sim.step(2)  # (the first step has nothing to diffuse)
        got.append((u, sim.get("i"), sim.get("u"), it, rr, st["it_diff"], st["it_elast"]))
        sim.close()
    a, b = got
    assert a[3] > 3 and max(a[5]) > 1
    assert a[3:] == b[3:]
    assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3]))
