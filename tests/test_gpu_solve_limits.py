"""Solves at the limits of what their entry points accept: the largest
iteration cap, very stiff or soft tissue, a tiny force, an indefinite
preconditioner."""
import ctypes

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


def _stiffer(k):
    """The workload's parameters with every modulus and the screening times 2^k: the displacement of the same
    force is that of k = 0 times 2^-k."""
    P = synthetic.params()
    for name in ("lame_scale", "eta_tumor", "eta_healthy", "eta_bg"):
        P[name] *= 2.0 ** k
    return P


@pytest.mark.parametrize("n", [16, 128, 256])
def test_mixed_solve_does_not_depend_on_the_unit_of_the_moduli(n):
    """Moduli 2^60 times as large.  The strains fit FP32 (about 1e-24 at 128^3), their squares do not.  The FP32
    vectors are the same numbers with another exponent, but for values under 2^-126 (1e-14 of the largest), so
    the iterations agree; one more is left to a residual that close to its threshold."""
    need_gpu()
    its = []
    for k in (0, 60):
        sim = _sim(n, "mixed", _stiffer(k))
        u, it, rr = sim.solve_elasticity()   # (an error if the FP64 residual misses rtol)
        sim.close()
        its.append(it)
        say(f"n={n}, moduli * 2^{k}: {it} iterations, residual {rr:.2e}, |u| {float(u.norm()):.3e}")
    assert abs(its[1] - its[0]) <= 1


# (grid, nu and E of the CSF, screening): a negative modulus that makes the mean material, and so the
# preconditioner, indefinite for the force, while the curvature along M^-1 r is positive
INDEFINITE = [(16, 0.441, -3997.0, 13597.0), (32, 0.4083, -5610.0, 22977.0), (64, 0.41811, -6532.7, 25278.0),
              (128, 0.4737, -1817.0, 261.0)]


# the same with a positive <r, M^-1 r> and a negative curvature
BREAKDOWN = [(16, 0.49, -500.0, 1e4), (128, 0.49, -700.0, 1e4), (256, 0.49, -700.0, 1e4)]


def _refused(n, nu, E, eta, precision):
    """Signs of <r, M^-1 r> and of the curvature along M^-1 r at the start of an elasticity solve that must end
    with TUMOR_ENAN before any iteration, the start vector unchanged."""
    torch = need_gpu()
    sim = _sim(n, precision, synthetic.params(nu_csf=nu, E_csf=E, eta_healthy=eta))
    b = -sim.apply_op("force", sim.get("p"))
    z = sim.apply_op("elast_precond", b)
    gamma, curv = float((b * z).sum()), float((z * sim.apply_op("elasticity", z)).sum())
    say(f"n={n} {precision}: <r, M^-1 r> = {gamma:.3e}, curvature {curv:.3e}")
    u, it, rr = torch.full((3, n, n, n), -1.0, dtype=torch.float64, device="cuda"), ctypes.c_int32(-1), ctypes.c_double(0)
    code = sim.lib.tumor_solve_elasticity(sim.ctx, None, tm._ptr(u), ctypes.byref(it), ctypes.byref(rr))
    sim.close()
    assert code == tm.ENAN
    assert it.value == 0 and not u.any()
    return gamma, curv


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,nu,E,eta", INDEFINITE)
def test_an_indefinite_preconditioner_is_refused_at_the_start(n, nu, E, eta, precision):
    gamma, curv = _refused(n, nu, E, eta, precision)
    assert gamma < 0.0 < curv


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,nu,E,eta", BREAKDOWN)
def test_a_negative_curvature_ends_the_solve(n, nu, E, eta, precision):
    gamma, curv = _refused(n, nu, E, eta, precision)
    assert curv < 0.0 < gamma


@pytest.mark.parametrize("k", [600, -600])
@pytest.mark.parametrize("n", [16, 64, 128, 256])
def test_fp64_solve_scales_exactly_with_the_moduli(n, k):
    """Powers of two are exact, so the solution is that of k = 0 times 2^-k, bit for bit, and its products and
    squares must all stay in range."""
    torch = need_gpu()
    got = []
    for e in (0, k):
        sim = _sim(n, "fp64", _stiffer(e))
        u, it, rr = sim.solve_elasticity()
        sim.close()
        say(f"n={n}, moduli * 2^{e}: {it} iterations, residual {rr:.2e}")
        got.append((u * 2.0 ** e, it, rr))
    assert got[0][1:] == got[1][1:]
    assert torch.equal(got[0][0], got[1][0])


@pytest.mark.parametrize("n", [16, 64, 128, 256])
def test_fp64_solve_of_a_tiny_force(n):
    """A random force of rms 2^-506: the per-mode products of the inner products, 1e-303 V at the start and 1e-16
    of that at the end, reach into the denormal range, with about six digits left at 16^3.  The largest terms
    decide alpha, so the count is that of the force of rms 1, give or take one."""
    torch = need_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    f = torch.randn((3, n, n, n), generator=gen, dtype=torch.float64, device="cuda")
    sim = _sim(n, "fp64", max_it=200)
    its = []
    for k in (0, -506):
        u, it, rr = sim.solve_elasticity(f * 2.0 ** k)   # (an error if it does not converge)
        say(f"n={n}, force * 2^{k}: {it} iterations, residual {rr:.2e}")
        its.append(it)
    sim.close()
    assert abs(its[1] - its[0]) <= 1
