"""The solves on every grid size their kernels are written for, against the
oracle: in iteration lockstep in FP64 (a few iterations, where every
operator, inner product and update counts), and by the FP64 residual of its
result in the mixed precision.

Tolerances: lockstep differs by rounding alone; a solve of k iterations of an
operator with condition number about 10 after preconditioning loses a few
digits of 1e-16, so 1e-11 leaves two orders.  The mixed form promises
||b - A u|| <= rtol ||b|| in FP64; 1.01 rtol allows for the oracle's own
rounding of the residual (1e-16 of ||A|| ||u||, under 1e-3 of rtol here).
"""
import ctypes

import numpy as np
import pytest

import paper_1810_05370_amd as tm
import synthetic
from gpu_common import need_gpu, rel_l2, say
from oracle import model, model_single
from oracle import reaction as rx
from oracle import solvers
from oracle.spectral import Grid, norm

pytestmark = pytest.mark.gpu


def _case(n, precision, rtol, max_it=1000):
    """A context with tumour, necrosis and a displacement to start from, and the oracle's system."""
    import torch
    inp = synthetic.workload_inputs("seeds3_n128", n=n)
    P = synthetic.params()
    sim = tm.from_inputs(inp, P, precision=precision, rtol_elast=rtol, max_it=max_it)
    rng = np.random.default_rng(3)
    u0 = np.stack([1e-3 * synthetic.random_field(n, 20 + a, 2.0) for a in range(3)])
    sim.set("u", torch.as_tensor(u0))
    nec = 0.1 * rng.random((n, n, n))
    sim.set("n", torch.as_tensor(nec))
    sim.refresh()
    p = sim.get("p").cpu().numpy()
    z = np.zeros_like(p)
    co = rx.refresh(P, p, z, nec, inp["gm"], inp["wm"], inp["csf"])
    g = Grid(n)
    return sim, g, co, rx.elastic_force(g, P["zeta"], p, nec), u0


@pytest.mark.parametrize("n", [16, 32, 64, 128, 256])
def test_elasticity_in_lockstep(n):
    need_gpu()
    its = 3 if n == 256 else 6
    say(f"elasticity lockstep n={n}, {its} iterations")
    # the iteration cap stops the solve; the last iterate is returned with ENOCONV
    sim, g, co, force, u0 = _case(n, "fp64", 1e-8, max_it=its)
    u, it, rr = sim.get("u"), ctypes.c_int32(0), ctypes.c_double(0)
    code = sim.lib.tumor_solve_elasticity(sim.ctx, None, tm._ptr(u), ctypes.byref(it), ctypes.byref(rr))
    it, rr = it.value, rr.value
    assert code == tm.ENOCONV
    ref, _, rr_ref, _ = solvers.solve_elasticity(g, co["mu"], co["lam"], co["eta"],
                                                 (co["mubar"], co["lambar"], co["etabar"]), force, u0, 1e-8, 100,
                                                 fixed_iters=its)
    err = rel_l2(u.cpu().numpy(), ref)
    say(f"  relL2 {err:.2e}, residual {rr:.3e} (oracle {rr_ref:.3e})")
    sim.close()
    assert it == its
    assert err < 1e-11
    assert abs(rr - rr_ref) <= 1e-9 * rr_ref


@pytest.mark.parametrize("n", [16, 32, 64, 128, 256])
def test_mixed_elasticity_meets_its_tolerance(n):
    need_gpu()
    say(f"mixed elasticity n={n}")
    sim, g, co, force, _ = _case(n, "mixed", 1e-8)
    u, it, rr = sim.solve_elasticity()
    res = -force - solvers.elasticity_op(g, co["mu"], co["lam"], co["eta"], u.cpu().numpy())
    rel = norm(res) / norm(force)
    say(f"  {it} iterations, residual {rr:.3e}, by the oracle {rel:.3e}")
    sim.close()
    assert it > 0 and rel <= 1.01e-8 and abs(rel - rr) <= 1e-10


@pytest.mark.parametrize("n", [16, 128, 256])
def test_diffusion_in_lockstep(n):
    """One species, so the solve is a batch of one: diffusion and reaction, three iterations."""
    need_gpu()
    say(f"diffusion lockstep n={n}")
    inp = synthetic.workload_inputs("seeds3_n128", n=n)
    P = synthetic.params()
    st = model.init_state(P, n, inp["wm"], inp["gm"], inp["csf"], inp["centers"], inp["sigmas"], inp["weights"])
    ref = model_single.step(st, dict(advection=False, elasticity=False), forced=[3, 0, 0, 0])
    sim = tm.from_inputs(inp, P, model="single", flags=0)
    sim.force_iterations([3, 0, 0, 0])
    got = sim.step(1)
    err = rel_l2(sim.get("p").cpu().numpy(), st.f["p"])
    rr, rr_ref = got["relres_diff"][0], ref["relres_diff"][0]
    say(f"  relL2 {err:.2e}, residual {rr:.3e} (oracle {rr_ref:.3e})")
    sim.close()
    assert got["it_diff"][0] == 3
    assert err < 1e-11
    # the residual after three iterations is a difference of terms about 1 / rr_ref
    # times its size, each rounded to 1e-16
    assert abs(rr - rr_ref) <= 1e-9 * rr_ref + 1e-13


def _three_systems(n, seed, **params):
    """Parameters, inputs and i, o, l in mid-simulation, each with its own spectrum (so its own iteration count)."""
    inp = synthetic.workload_inputs("seeds3_n128", n=n)
    fields = dict(i=0.3 * synthetic.random_field(n, seed, 1.0) ** 2, o=0.8 + 0.02 * synthetic.random_field(n, seed + 1, 2.0),
                  l=0.05 * synthetic.random_field(n, seed + 2, 0.5) ** 2)
    return synthetic.params(**params), inp, fields


@pytest.mark.parametrize("forced", [(2, 4, 3), (3, 0, 5)])
@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_batched_diffusion_in_lockstep(n, forced):
    """i, o and l as one batch; each ends at its own launch, or takes no part."""
    import torch
    need_gpu()
    say(f"batched diffusion lockstep n={n}, iterations {forced}")
    P, inp, fields = _three_systems(n, 40)
    st = model.init_state(P, n, inp["wm"], inp["gm"], inp["csf"], inp["centers"], inp["sigmas"], inp["weights"])
    st = model.State(st.grid, P, dict(st.f, **fields), st.u, st.u_prev)
    ref = model.step(st, dict(advection=False, elasticity=False), forced=[*forced, 0])
    sim = tm.from_inputs(inp, P, flags=tm.F_EDEMA)
    for k, v in fields.items():
        sim.set(k, torch.as_tensor(v))
    sim.refresh()
    sim.force_iterations([*forced, 0])
    got = sim.step(1)
    err = {k: rel_l2(sim.get(k).cpu().numpy(), st.f[k]) for k in ("p", "i", "o", "l")}
    say(f"  relL2 {err}, residuals {got['relres_diff']} (oracle {ref['relres_diff']})")
    sim.close()
    assert tuple(got["it_diff"]) == forced
    assert max(err.values()) < 1e-11
    for rr, rr_ref in zip(got["relres_diff"], ref["relres_diff"]):
        assert abs(rr - rr_ref) <= 1e-9 * rr_ref + 1e-13


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [32, 128])
def test_batched_diffusion_meets_its_tolerance(n, precision):
    """With every reaction rate zero a step leaves the solutions of the three systems in i, o and l."""
    import torch
    need_gpu()
    rates = ("rho_w", "rho_g", "alpha0", "beta0", "gamma", "delta_s", "delta_p", "delta_e", "delta_l")
    P, inp, fields = _three_systems(n, 50, **{k: 0.0 for k in rates})
    sim = tm.from_inputs(inp, P, precision=precision, flags=tm.F_EDEMA)
    for k, v in fields.items():
        sim.set(k, torch.as_tensor(v))
    sim.refresh()
    got = sim.step(1)
    g, K = Grid(n), P["k_w"] * inp["wm"] + P["k_g"] * inp["gm"] + P["k_f"] * inp["csf"]
    rel = []
    for k in ("i", "o", "l"):
        rhs = solvers.cn_rhs(g, K, 0.01, fields[k])
        rel.append(norm(rhs - solvers.cn_matrix(g, K, 0.01, sim.get(k).cpu().numpy())) / norm(rhs))
    say(f"batched diffusion n={n} {precision}: {got['it_diff']} iterations, residuals {got['relres_diff']}, by the oracle {rel}")
    sim.close()
    assert min(got["it_diff"]) < max(got["it_diff"])
    for a, b in zip(rel, got["relres_diff"]):
        assert a <= 1.01e-8 and abs(a - b) <= 1e-10


@pytest.mark.parametrize("n", [32, 64])
def test_one_diffusion_system_in_lockstep(n):
    need_gpu()
    say(f"one diffusion system n={n}")
    inp = synthetic.workload_inputs("seeds3_n128", n=n)
    P = synthetic.params()
    st = model.init_state(P, n, inp["wm"], inp["gm"], inp["csf"], inp["centers"], inp["sigmas"], inp["weights"])
    ref = model_single.step(st, dict(advection=False, elasticity=False), forced=[4, 0, 0, 0])
    sim = tm.from_inputs(inp, P, model="single", flags=0)
    sim.force_iterations([4, 0, 0, 0])
    got = sim.step(1)
    err = rel_l2(sim.get("p").cpu().numpy(), st.f["p"])
    rr, rr_ref = got["relres_diff"][0], ref["relres_diff"][0]
    say(f"  relL2 {err:.2e}, residual {rr:.3e} (oracle {rr_ref:.3e})")
    sim.close()
    assert got["it_diff"][0] == 4
    assert err < 1e-11
    assert abs(rr - rr_ref) <= 1e-9 * rr_ref + 1e-13


def test_elasticity_at_512_meets_its_tolerance():
    """Random tissue (every mode takes part), both precisions.  The residual is taken by the FP64 operator of the
    unfused passes, which test_gpu_maxsize.py checks on plane waves, so none of the solves' fused kernels judges
    itself.  Its rounding, about 1e-16 of ||A|| ||u||, stays under 1e-10 of ||f||."""
    torch = need_gpu()
    n = 512
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    w = 0.3 + 0.4 * torch.rand((n, n, n), generator=gen, dtype=torch.float64, device="cuda")
    g = 0.1 + 0.1 * torch.rand((n, n, n), generator=gen, dtype=torch.float64, device="cuda")
    c = 1.0 - w - g
    centers, sigmas, weights = synthetic.tumor_seeds("three", 1)
    sols = {}
    for precision in ("mixed", "fp64"):
        sim = tm.Tumor(n, synthetic.params(), w, g, c, centers, sigmas, weights, precision=precision)
        say(f"512^3 elasticity, {precision}")
        sols[precision] = sim.solve_elasticity()
        say(f"  {sols[precision][1]} iterations, residual {sols[precision][2]:.3e}")
        if precision == "mixed":
            sim.close()
            del sim
            torch.cuda.empty_cache()
    f = sim.apply_op("force", sim.get("p") + sim.get("n"))
    for precision, (u, it, rr) in sols.items():
        rel = float((f + sim.apply_op("elasticity", u)).norm() / f.norm())
        say(f"  {precision}: by the unfused operator {rel:.3e}")
        assert it > 5
        assert rel <= 1.01e-8 and abs(rel - rr) <= 1e-10
    sim.close()


@pytest.mark.parametrize("n", [256, 512])
def test_batched_diffusion_of_large_grids_meets_its_tolerance(n):
    """As test_batched_diffusion_meets_its_tolerance, judged on the device by the FP64 operator of the unfused
    passes with the coefficients the solve had."""
    torch = need_gpu()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)

    def rand(lo, hi):
        return lo + (hi - lo) * torch.rand((n, n, n), generator=gen, dtype=torch.float64, device="cuda")
    w, g = rand(0.3, 0.7), rand(0.1, 0.2)
    x = torch.arange(n, dtype=torch.float64, device="cuda") * (2.0 * np.pi / n)
    # (a smooth field, a rough one and one in between: three iteration counts)
    fields = dict(i=rand(0.0, 0.3), o=0.8 + 0.1 * torch.cos(3.0 * x) * torch.ones_like(w),
                  l=0.05 + 0.01 * torch.cos(9.0 * x)[:, None, None] + rand(0.0, 1e-4))
    rates = ("rho_w", "rho_g", "alpha0", "beta0", "gamma", "delta_s", "delta_p", "delta_e", "delta_l")
    P = synthetic.params(**{k: 0.0 for k in rates})
    sols = {}
    for precision in ("mixed", "fp64"):
        sim = tm.Tumor(n, P, w, g, 1.0 - w - g, precision=precision, flags=tm.F_EDEMA)
        for k, v in fields.items():
            sim.set(k, v)
        sim.refresh()
        st = sim.step(1)
        say(f"batched diffusion {n}^3 {precision}: {st['it_diff']} iterations, residuals {st['relres_diff']}")
        sols[precision] = (st, [sim.get(k) for k in fields])
        if precision == "mixed":
            sim.close()
            del sim
            torch.cuda.empty_cache()
    sim.set("w", w)
    sim.set("g", g)
    sim.refresh()
    for precision, (st, out) in sols.items():
        rel = []
        for x0, x1 in zip(fields.values(), out):
            rhs = x0 + 0.005 * sim.apply_op("diffusion", x0)
            rel.append(float((rhs - x1 + 0.005 * sim.apply_op("diffusion", x1)).norm() / rhs.norm()))
        say(f"  {precision}: by the unfused operator {rel}")
        assert min(st["it_diff"]) < max(st["it_diff"])
        for a, b in zip(rel, st["relres_diff"]):
            assert a <= 1.01e-8 and abs(a - b) <= 1e-10
    sim.close()
