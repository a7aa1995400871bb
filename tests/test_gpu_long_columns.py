"""Columns of more than 2^16 + 1 nodes: grids of 17 levels and more.

Two V-cycles against the oracle (1e-12, as for every V-cycle) and a step in
mixed precision to the rounding floor (1e-10); the sink's root density and the
Remark's shift are per-level data.
"""
import dataclasses

import pytest

import oracle
import paper_2606_04292_amd as rsl
from tests.test_gpu_parity import FLOOR_CYCLES, TOL_CONV, TOL_SWEEP, np_, rel, say
from tests.test_gpu_wg_cycle import D, F, N, REMARK, SINK, VG, _box

pytestmark = pytest.mark.gpu

CASES = {
    "131073": _box([131073], VG, [F, N], [0.0, 0.0]),
    "131073_sink": _box([131073], SINK, [N, N], [0.0, 0.0]),
    "131073_remark": _box([131073], REMARK, [D, N], [-1.0, 0.0]),
    "262145": _box([262145], VG, [D, D], [-1.0, -0.5]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vcycles_match_the_oracle(name):
    w = CASES[name]
    S = oracle.Solver(w, oracle.ORDER_RB)
    G = rsl.Grid(w)
    say("long column", name, "levels", G.nlev)
    assert G.nlev == S.nlev == w.grid.levels()
    S.begin_step()
    G.begin_step()
    for c in range(2):
        S.vcycle()
        G.vcycle()
        e = rel(np_(G.psi()), S.psi())
        say("  cycle", c, "rel", e)
        assert e <= TOL_SWEEP, (name, c, e)
    G.close()


def test_mixed_step_matches_fp64():
    """On such a column a step's FP64 and mixed solutions agree at the rounding floor."""
    w = dataclasses.replace(CASES["131073"], dt=1e-6)
    got = []
    for precision in (rsl.RS_FP64, rsl.RS_MIXED):
        G = rsl.Grid(w, precision=precision)
        code, st = G.bdf_step(opts=rsl.solve_opts(2, 2, 32, max_cycles=FLOOR_CYCLES, tol_abs=0.0,
                                                  stagnation=1))
        assert code == rsl.RS_OK, rsl.lib().rs_last_error()
        got.append(np_(G.get_state()[0]))
        say("long column, step", precision, "cycles", st.cycles)
        G.close()
    assert rel(got[1], got[0]) <= TOL_CONV
