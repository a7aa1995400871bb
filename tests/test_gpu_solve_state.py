"""A pointwise solve starts from the node's value and nothing else.

What a solve returns does not depend on earlier sweeps, visits or cycles, so a
batch of sweeps is bit for bit that many single sweeps, the sweeps of a level
in one work-group are those of one launch per colour, and the cycles of a step
in one launch are those of that many V-cycle calls.  Each node's arithmetic is
the same sequence of roundings on every one of these routes, hence equality
without a tolerance.
"""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2606_04292_amd as rsl
from tests.test_gpu_parity import np_, say
from tests.test_gpu_wg_cycle import CASES

pytestmark = pytest.mark.gpu


def _same(name, a, b):
    d = np.count_nonzero(a != b)
    say("bits", name, "values that differ:", d, "of", a.size)
    assert d == 0


def _swept(w, batches):
    G = rsl.Grid(w)
    G.begin_step()
    for n in batches:
        G.sweep(n)
    x = np_(G.psi())
    G.close()
    return x


@pytest.mark.parametrize("name", ["1d_127_slots", "1d_2049_all_unknown", "1d_1025_sink",
                                  "2d_33x33", "2d_129x9_remark", "3d_5x5x5", "3d_17x17x5",
                                  "soils_33", "soils_1025"])
def test_a_batch_of_sweeps_is_that_many_single_sweeps(name):
    _same(name, _swept(CASES[name], [60]), _swept(CASES[name], [1] * 60))


# levels of more than 1024 nodes, which RS_SWEEP keeps with the launched sweeps
@pytest.mark.parametrize("name", ["1d_2049_all_unknown", "1d_1025_sink", "2d_33x33", "2d_257x5",
                                  "2d_129x9_remark", "3d_17x17x5", "3d_9x9x17_sink",
                                  "soils_33", "soils_1025"])
def test_sweeps_in_one_work_group_are_those_of_colour_launches(name, monkeypatch):
    here = _swept(CASES[name], [7])
    monkeypatch.setenv("RS_SWEEP", "single")
    _same(name, here, _swept(CASES[name], [7]))


# 70 cycles cross the end of a launch of the whole-grid solve
@pytest.mark.parametrize("cycles", [9, 70])
@pytest.mark.parametrize("name", ["1d_127_slots", "1d_1025_sink", "2d_33x33", "2d_257x5",
                                  "3d_5x5x5", "3d_9x9x17_sink", "soils_33"])
def test_the_cycles_of_a_step_are_those_of_vcycle_calls(name, cycles):
    w = CASES[name]
    G = rsl.Grid(w)
    code, st = G.bdf_step(opts=rsl.solve_opts(w.nu1, w.nu2, 32, max_cycles=cycles, tol_abs=0.0))
    # (a defect of exactly zero ends the step before)
    done = st.cycles
    x = np_(G.psi() if code == rsl.RS_ENOTCONV else G.get_state()[0])
    if code == rsl.RS_ENOTCONV:   # the norm reported is that of the iterate left
        assert st.res == G.residual_norm()
    assert (code == rsl.RS_ENOTCONV and done == cycles) or (code == rsl.RS_OK and st.res == 0.0)
    G.close()
    G = rsl.Grid(w)
    G.begin_step()
    for _ in range(done):
        G.vcycle()
    _same("%s, %d cycles" % (name, done), x, np_(G.psi()))
    G.close()


@pytest.mark.parametrize("name", ["1d_127_slots", "1d_1025_sink", "2d_33x33", "3d_5x5x5", "soils_33"])
def test_the_stopping_test_crosses_launches(name):
    """So many sweeps on the coarsest level are allowed that a launch of the whole-grid solve
    holds two cycles: the step ends where the stopping rule ends V-cycle calls."""
    w = CASES[name]
    G = rsl.Grid(w)
    code, st = G.bdf_step(opts=rsl.solve_opts(w.nu1, w.nu2, 3000, max_cycles=100, tol_abs=0.0,
                                              stagnation=1))
    assert code == rsl.RS_OK, rsl.lib().rs_last_error()
    x = np_(G.get_state()[0])
    # the same cycles one by one (the coarsest level's sweeps stay as set by the step)
    G.set_state(torch.as_tensor(w.psi0))
    G.begin_step()
    best, slow, hist = G.residual_norm(), 0, []
    while slow < 2:
        hist.append(G.vcycle(want_norm=True))
        if hist[-1] == 0.0:
            break
        best, slow = (hist[-1], 0) if hist[-1] < best else (best, slow + 1)
    say("launches", name, "cycles", st.cycles, len(hist))
    assert st.cycles == len(hist) and list(st.res_hist[1:1 + len(hist)]) == hist[:63]
    _same(name, x, np_(G.psi()))
    G.close()
