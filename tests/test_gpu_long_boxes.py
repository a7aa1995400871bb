"""3-D levels of more nodes per colour than the one-work-group cycle has threads.

5x5x65 nodes in each order of the axes, as a grid and as the second level of
9x9x129: two nodes per thread and colour.  Two V-cycles against the oracle
(1e-12, as for every V-cycle) and two steps to the rounding floor in FP64 and
mixed precision (1e-10).
"""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2606_04292_amd as rsl
from paper_2606_04292_amd import workloads as W
from tests.test_gpu_parity import FLOOR_CYCLES, TOL_CONV, TOL_SWEEP, np_, rel, say
from tests.test_gpu_wg_cycle import D, F, HK, N, SINK, VG, _box

pytestmark = pytest.mark.gpu


def _soils(n):
    w = W.two_layer_vg(33)
    g = _box(n, w.law, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]).grid
    ids = (np.arange(np.prod(g.shape)) % len(w.soils)).astype(np.uint8).reshape(g.shape)
    return dataclasses.replace(w, grid=g, soil_id=ids, psi0=_box(n, VG, [N] * 6, [0.0] * 6).psi0)


CASES = {
    "5x5x65": _box([5, 5, 65], VG, [N] * 4 + [F, N], [0.0] * 6),
    "5x65x5": _box([5, 65, 5], SINK, [N] * 6, [0.0] * 6),
    "65x5x5": _box([65, 5, 5], HK, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0],
                   patch=(2, (20, 1), (44, 3))),
    "9x9x129": _box([9, 9, 129], VG, [D, N, N, N, N, D], [-1.0, 0, 0, 0, 0, -0.6]),
    "soils_5x5x65": _soils([5, 5, 65]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_vcycles_match_the_oracle(name):
    w = CASES[name]
    say("long box", name)
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


@pytest.mark.parametrize("precision", [rsl.RS_FP64, rsl.RS_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(n for n in CASES if not n.startswith("soils")))
def test_steps_match_the_oracle(name, precision):
    w = CASES[name]
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
        say("  step", name, precision, step, "corrections", st.cycles, "rel", e)
        assert e <= TOL_CONV, (name, step, e)
    G.close()
