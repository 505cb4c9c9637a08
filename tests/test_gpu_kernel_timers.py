"""The kernel timers' launches and algorithmic bytes, counted by hand for the
three kinds of Krylov iteration: every array a kernel reads or writes once,
every launch of a solve in some class.  All of them are whole numbers, so
nothing is left to a tolerance."""
import pytest

import paper_1810_05370_amd as tm
import synthetic
from gpu_common import need_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 128, 256])
def test_an_elasticity_solve_is_timed_whole(n):
    need_gpu()
    classes = ("krylov64", "xelast64", "zinvp64", "coldot64", "tileinv64", "tilex64", "tilefwd64")
    sim = tm.from_inputs(synthetic.workload_inputs("seeds3_n128", n=n), synthetic.params())
    for c in classes:
        sim.kernel_timer(c, True)
    _, it, _ = sim.solve_elasticity()
    got = {c: sim.kernel_timer_read(c) for c in classes}
    sim.close()
    A = 8 * n ** 3  # one array
    # the residual at the start: x, b and A x in three components; its operator's x pass
    want = {c: [0, 0] for c in classes}
    want["krylov64"], want["xelast64"] = [1, 9 * A], [1, 19 * A]

    def add(c, launches, nbytes):
        want[c][0] += launches
        want[c][1] += launches * nbytes

    if n <= 64:
        add("krylov64", 1, 7 * A)        # start: the residual, r, the preconditioner
        add("krylov64", 1, 6 * A)        # coefficients turned
        add("zinvp64", it, 14 * A)
        add("xelast64", it, 19 * A)
        add("krylov64", it, 35 * A)
        add("krylov64", 1, 9 * A)        # x64 += x
    elif n == 256:
        add("krylov64", 1, 12 * A)       # start: the residual; r, p, x
        add("tileinv64", 1, 12 * A)
        add("tileinv64", it - 1, 24 * A)
        add("tilex64", it, 20 * A)
        add("tilefwd64", it, 14 * A)
        add("krylov64", it, 16 * 16 * (n // 2 // 2))     # scalars: two sums of each tile of 2 columns
        add("krylov64", 1, 12 * A)       # x64 += x + alpha p
    else:
        add("krylov64", 1, 6 * A)        # start: r, p
        add("zinvp64", it - 1, 21 * A)
        add("xelast64", it, 19 * A)
        add("coldot64", it, 12 * A)
        add("krylov64", it, 16 * n * (n // 2 // 16))     # scalars: two sums of each tile of 16 columns
        add("krylov64", 1, 9 * A)        # x += alpha p
    for c in classes:
        say(f"n={n} {c}: {got[c]}, by hand {want[c]}")
    assert it > 10
    for c in classes:
        assert [got[c]["launches"], got[c]["bytes"]] == want[c], c


@pytest.mark.parametrize("n", [64, 128])
def test_batched_diffusion_timers_count_each_system_while_it_iterates(n):
    """Mixed: system k iterates it_diff[k] times in outer_diff[k] solves.  Per system and iteration the first
    pass moves 5 arrays up to 64^3, 7 above (3 in a solve's first iteration, which takes p as it is), the x pass
    6 with K once per launch, the last pass (above 64^3) 5."""
    need_gpu()
    sim = tm.from_inputs(synthetic.workload_inputs("seeds3_n128", n=n), synthetic.params(), precision="mixed")
    sim.step(3)   # i and l nonzero: all three systems iterate
    classes = ("zinvpb32", "xdiff32", "coldot32")
    for c in classes:
        sim.kernel_timer(c, True)
    st = sim.step(1)
    got = {c: sim.kernel_timer_read(c) for c in classes}
    sim.close()
    say(f"n={n}: {got}, iterations {st['it_diff']}, solves {st['outer_diff']}, elasticity {st['it_elast']}")
    its, outer = sum(st["it_diff"]), sum(st["outer_diff"])
    A = 4 * n ** 3
    assert min(st["it_diff"]) < max(st["it_diff"])
    assert got["zinvpb32"]["bytes"] == A * (5 * its if n <= 64 else 7 * its - 4 * outer)
    assert got["xdiff32"]["bytes"] == A * (6 * its + got["xdiff32"]["launches"])
    assert got["xdiff32"]["launches"] == got["zinvpb32"]["launches"]
    # (the elasticity's last pass is in the same class: 12 arrays)
    assert got["coldot32"]["bytes"] == (0 if n <= 64 else A * (5 * its + 12 * st["it_elast"]))
