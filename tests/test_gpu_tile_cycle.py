"""The tiled mid-size levels (1-D, 2-D) at the edges of their tile shapes.

Two V-cycles against the oracle (1e-12, as for every V-cycle), an FMG cycle,
and mixed-precision steps to the rounding floor against the FP64 oracle
(1e-10).  Shapes: square levels with several tiles, levels whose short axis is
loaded whole, the largest tiled level and the first one above it; smoothing
counts that fit one launch (1, 2, 3), need three (5, 10), and none at all;
Dirichlet faces, a patch, free drainage, a sink, the Remark's shift, per-node
soils, values from the state.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2606_04292_amd as rsl
from paper_2606_04292_amd import workloads as W
from tests.test_gpu_parity import FLOOR_CYCLES, TOL_CONV, TOL_SWEEP, np_, rel, say
from tests.test_gpu_wg_cycle import D, F, HK, N, REMARK, SINK, VG, _box

pytestmark = pytest.mark.gpu


def _nu(w, nu1, nu2=None):
    return dataclasses.replace(w, nu1=nu1, nu2=nu1 if nu2 is None else nu2)


CASES = {
    "65x65_nu1": _nu(_box([65, 65], VG, [N, N, F, N], [0.0] * 4, patch=(3, (20, 0), (44, 0))), 1),
    "129x65_nu2": _box([129, 65], VG, [N, N, F, N], [0.0] * 4, patch=(1, (17, 0), (30, 0))),
    "65x129_nu3": _nu(_box([65, 129], HK, [D, N, D, N], [-1.0, 0, -0.8, 0.0]), 3),
    "129x129_nu5_0": _nu(_box([129, 129], VG, [N, D, N, N], [0.0, -0.7, 0.0, 0.0]), 5, 0),
    "65x65_nu0_10": _nu(_box([65, 65], VG, [N, D, N, D], [0.0, -0.7, 0.0, -0.9]), 0, 10),
    "65x65_nu23": _nu(_box([65, 65], VG, [N, D, N, D], [0.0, -0.7, 0.0, -0.9]), 23, 4),
    "513x9": _box([513, 9], VG, [N, N, D, N], [0, 0, -0.8, 0.0]),
    "5x1025_sink": _box([5, 1025], SINK, [N] * 4, [0.0] * 4),
    "3x2049": _box([3, 2049], VG, [N, N, D, D], [0, 0, -0.8, -0.5]),
    "65x65_remark": _box([65, 65], REMARK, [D, N, D, N], [-1.0, 0, -0.8, 0.0]),
    "513x257": _box([513, 257], VG, [N, N, D, N], [0, 0, -0.8, 0.0]),
    "4097": _box([4097], VG, [F, N], [0.0, 0.0]),
    "8193_nu5": _nu(_box([8193], HK, [D, D], [-1.0, -0.5]), 5),
    "soils_65_nu10": W.two_layer_vg(65),
    "gardner_65_nu5": W.gardner_2d(65),
    "state_top_129": dataclasses.replace(
        _box([129, 129], VG, [N, N, D, W.BC_DIRICHLET_STATE], [0, 0, -0.8, 0.0]), nu1=2),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vcycles_match_the_oracle(name):
    w = CASES[name]
    say("tiles", name, w.grid.n, w.nu1, w.nu2)
    for mode in ("vcycle", "fmg"):
        S = oracle.Solver(w, oracle.ORDER_RB)
        G = rsl.Grid(w)
        S.begin_step()
        G.begin_step()
        for c in range(2 if mode == "vcycle" else 1):
            getattr(S, mode)()
            getattr(G, mode)()
            e = rel(np_(G.psi()), S.psi())
            say("  %s %d rel" % (mode, c), e)
            assert e <= TOL_SWEEP, (name, mode, c, e)
        G.close()


STEPS = ["65x65_nu1", "129x65_nu2", "65x129_nu3", "65x65_nu23", "5x1025_sink", "3x2049", "4097"]


@pytest.mark.parametrize("precision", [rsl.RS_FP64, rsl.RS_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", STEPS)
def test_steps_match_the_oracle(name, precision):
    w = CASES[name]
    say("tiles, steps", name, precision)
    S = oracle.Solver(w, oracle.ORDER_RB)
    G = rsl.Grid(w, precision=precision)
    opts = rsl.solve_opts(w.nu1, w.nu2, w.nu_coarse, max_cycles=FLOOR_CYCLES, tol_abs=0.0,
                          stagnation=1, mp_inner_cycles=2)
    for step in range(2):
        S.begin_step()
        oracle.solve_to_floor(S, FLOOR_CYCLES, 0.0)
        S.end_step()
        code, st = G.bdf_step(opts=opts)
        assert code == rsl.RS_OK, rsl.lib().rs_last_error()
        e = rel(np_(G.get_state()[0]), S.get(oracle.FIELD_PSI_N))
        say("  step", step, "cycles", st.cycles, "rel", e)
        assert e <= TOL_CONV, (name, step, e)
    G.close()


def test_step_out_of_cycles_keeps_the_smoothed_iterate():
    """A step that runs out of cycles ends on the pre-smoothed iterate its last norm was taken
    on, also where the next coarse part was queued ahead: the same state as smoothing plainly."""
    w = CASES["129x65_nu2"]
    G = rsl.Grid(w)
    code, st = G.bdf_step(opts=rsl.solve_opts(2, 2, 32, max_cycles=3, tol_abs=0.0))
    assert code == rsl.RS_ENOTCONV and st.cycles == 3
    norm = G.residual_norm()
    assert abs(norm - st.res) <= 1e-10 * st.res0
    S = oracle.Solver(w, oracle.ORDER_RB)
    S.begin_step()
    S.vcycle()
    S.vcycle()
    S.sweep(2, 0)
    e = rel(np_(G.psi()), S.psi())
    say("out of cycles: rel", e, "norm", norm, st.res)
    assert e <= TOL_SWEEP
    G.close()
