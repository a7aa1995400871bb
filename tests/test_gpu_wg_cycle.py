"""The one-work-group cycle on the level sizes where its slot maps turn over.

Two V-cycles of grids that run wholly (or from their first coarse level) in
one work-group, against the oracle (1e-12, as for every V-cycle), and for the
laws the FP32 cycle serves two mixed-precision steps to the rounding floor
against the FP64 oracle (1e-10).  Shapes: 64 / 65 nodes of one colour (one
wave / work-group barriers), the largest 1-D level with every node unknown
(1025 red nodes, two per thread), 2-D and 3-D levels up to the work-group's
two nodes per thread and the first shape above it, unequal axes, the smallest
grids; Dirichlet faces, a patch, sinks, the Remark's shift and per-node soils.
"""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2606_04292_amd as rsl
from paper_2606_04292_amd import workloads as W
from tests.test_gpu_parity import FLOOR_CYCLES, TOL_CONV, TOL_SWEEP, np_, rel, say

pytestmark = pytest.mark.gpu


def _box(n, law, bc, value, patch=None):
    h = 1.0 / (max(n) - 1)
    g = W.GridSpec(dim=len(n), n=list(n), L=[h * (m - 1) for m in n], face_bc=bc, face_value=value)
    if patch:
        g = dataclasses.replace(g, patch_face=patch[0], patch_lo=patch[1], patch_hi=patch[2],
                                patch_value=-0.05)
    x = np.zeros(g.shape)
    for a, m in enumerate(g.shape):
        sh = [1] * g.dim
        sh[a] = m
        x = x + np.cos(2.0 * np.linspace(0.0, 1.0, m) + a).reshape(sh)
    return W.Workload("box", g, law, -1.2 + 0.25 * x, dt=60.0, steps=2, order=2)


N, D, F = W.BC_NOFLUX, W.BC_DIRICHLET, W.BC_FREEDRAIN
VG = dataclasses.replace(W.config1(5).law, newton_tol=1e-10, xi=1e-6)
HK = W.config3(5).law
SINK = W.config4(5, 5).law
REMARK = dataclasses.replace(VG, kappa_rule=W.KAPPA_REMARK)

CASES = {
    "1d_3": _box([3], VG, [D, D], [-1.0, -0.5]),
    "1d_127_slots": _box([129], VG, [N, N], [0.0, 0.0]),
    "1d_2049_all_unknown": _box([2049], VG, [F, N], [0.0, 0.0]),
    "1d_1025_sink": _box([1025], SINK, [N, N], [0.0, 0.0]),
    "2d_33x33": _box([33, 33], VG, [N, N, F, N], [0.0] * 4, patch=(3, (10, 0), (21, 0))),
    "2d_257x5": _box([257, 5], HK, [N, N, D, N], [0, 0, -0.8, 0.0]),
    "2d_129x9_remark": _box([129, 9], REMARK, [D, N, D, N], [-1.0, 0, -0.8, 0.0]),
    "2d_65x65": _box([65, 65], VG, [N, D, N, N], [0.0, -0.7, 0.0, 0.0]),
    "3d_3x3x3": _box([3, 3, 3], HK, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
    "3d_5x5x5": _box([5, 5, 5], VG, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
    "3d_9x9x17_sink": _box([9, 9, 17], SINK, [N] * 6, [0.0] * 6),
    "3d_17x17x5": _box([17, 17, 5], HK, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0],
                       patch=(0, (3, 1), (9, 3))),
    "3d_9x33x9": _box([9, 33, 9], VG, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
    "soils_33": W.two_layer_vg(33),
    "soils_1025": W.celia_composite(1025),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vcycles_match_the_oracle(name):
    w = CASES[name]
    say("wg cycle", name, w.grid.n)
    S = oracle.Solver(w, oracle.ORDER_RB)
    G = rsl.Grid(w)
    S.begin_step()
    G.begin_step()
    for c in range(2):
        S.vcycle()
        G.vcycle()
        e = rel(np_(G.psi()), S.psi())
        say("  cycle", c, "rel", e)
        assert e <= TOL_SWEEP, (name, c, e)
    G.close()


@pytest.mark.parametrize("name", sorted(CASES))
def test_sweeps_of_one_level_match_the_oracle(name):
    """Sweeps on their own (one launch in one work-group where the level fits
    it), an odd number and a second batch, on the finest and coarsest level."""
    w = CASES[name]
    say("wg sweeps", name, w.grid.n)
    S = oracle.Solver(w, oracle.ORDER_RB)
    G = rsl.Grid(w)
    S.begin_step()
    G.begin_step()
    for lev in sorted({0, S.nlev - 1}):
        for f in ("PSI", "KSTAR", "G"):
            G.set_field(getattr(rsl, "FIELD_" + f),
                        torch.as_tensor(S.get(getattr(oracle, "FIELD_" + f), lev)), lev)
        for n in (3, 2):
            S.sweep(n, lev)
            G.sweep(n, lev)
            e = rel(np_(G.psi(lev)), S.psi(lev))
            say("  level", lev, "sweeps", n, "rel", e)
            assert e <= TOL_SWEEP, (name, lev, n, e)
    G.close()


@pytest.mark.parametrize("precision", [rsl.RS_FP64, rsl.RS_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(n for n in CASES if not n.startswith("soils")))
def test_steps_match_the_oracle(name, precision):
    """FP64: the step's cycles and its stopping test run in one launch on these grids."""
    w = CASES[name]
    if w.law.kappa_rule == W.KAPPA_REMARK:
        w = dataclasses.replace(w, steps=1)
    say("wg cycle, steps", name, precision)
    S = oracle.Solver(w, oracle.ORDER_RB)
    G = rsl.Grid(w, precision=precision)
    opts = rsl.solve_opts(w.nu1, w.nu2, w.nu_coarse, max_cycles=FLOOR_CYCLES, tol_abs=0.0,
                          stagnation=1)
    for step in range(w.steps):
        S.begin_step()
        oracle.solve_to_floor(S, FLOOR_CYCLES, 0.0)
        S.end_step()
        code, st = G.bdf_step(opts=opts)
        assert code == rsl.RS_OK, rsl.lib().rs_last_error()
        e = rel(np_(G.get_state()[0]), S.get(oracle.FIELD_PSI_N))
        say("  step", step, "corrections", st.cycles, "rel", e)
        assert e <= TOL_CONV, (name, step, e)
    G.close()


@pytest.mark.parametrize("name", ["1d_127_slots", "3d_5x5x5", "soils_33"])
def test_solve_in_several_launches(name):
    """More cycles than one launch of the whole-grid solve runs, without a tolerance to reach:
    as many cycles as asked for, the reported norms are those of the iterates."""
    w = CASES[name]
    G = rsl.Grid(w)
    code, st = G.bdf_step(opts=rsl.solve_opts(w.nu1, w.nu2, 32, max_cycles=130, tol_abs=0.0))
    if code == rsl.RS_OK:       # a defect of exactly zero ends the step
        assert st.res == 0.0
    else:
        assert code == rsl.RS_ENOTCONV and st.cycles == 130 and st.n_hist == 64
    G.set_state(G.torch.as_tensor(w.psi0))
    G.begin_step()
    r0 = G.residual_norm()
    assert abs(st.res0 - r0) <= 1e-12 * r0 and st.res_hist[0] == st.res0
    G.vcycle()
    r1 = G.residual_norm()
    say("several launches", name, st.cycles, st.res, "first cycle", st.res_hist[1], r1)
    assert abs(st.res_hist[1] - r1) <= 1e-9 * r0
    G.close()
