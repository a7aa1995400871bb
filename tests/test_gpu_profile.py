"""Profiling changes nothing but the clocks.

With the profile on, the finest level of a tiled grid smooths in launches of
its own (they are timed) while the levels below keep their kernels; the per-node
arithmetic is the same on both routes, so the iterates are equal bit for bit.
"""
import dataclasses

import numpy as np
import pytest

import paper_2606_04292_amd as rsl
from tests.test_gpu_parity import np_, say
from tests.test_gpu_tile_cycle import CASES
from tests.test_gpu_wg_cycle import D, N, VG, _box

pytestmark = pytest.mark.gpu

GRIDS = {
    "129x65": CASES["129x65_nu2"],
    "4097": CASES["4097"],
    "5x2049": _box([5, 2049], VG, [N, N, D, D], [0, 0, -0.8, -0.5]),
    "65x65x17": _box([65, 65, 17], VG, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
}


@pytest.mark.parametrize("precision", [rsl.RS_FP64, rsl.RS_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_profile_on_gives_the_same_cycles_and_steps(name, precision):
    w = dataclasses.replace(GRIDS[name], order=2)
    got = []
    for prof in (False, True):
        G = rsl.Grid(w, precision=precision)
        G.profile_enable(prof)
        G.begin_step()
        for _ in range(2):
            if precision == rsl.RS_FP64:
                G.vcycle()
            else:
                G.correction_cycle(2)
        cycles = np_(G.psi())
        G.fmg()
        fmg = np_(G.psi())
        G.set_state(G.torch.as_tensor(w.psi0))
        code, st = G.bdf_step(opts=rsl.solve_opts(w.nu1, w.nu2, 32, max_cycles=60, tol_abs=0.0,
                                                  stagnation=1))
        assert code == rsl.RS_OK, (prof, rsl.lib().rs_last_error())
        got.append((cycles, fmg, np_(G.get_state()[0]), st.cycles))
        # switched off again, the next cycle is an unprofiled one
        G.profile_enable(False)
        G.begin_step()
        G.vcycle()
        got[-1] += (np_(G.psi()),)
        G.close()
    say("profile", name, precision, "cycles of the step", got[0][3], got[1][3])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
