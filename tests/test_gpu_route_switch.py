"""The sweep switch set and cleared between calls on one grid.

RS_SWEEP sends a grid's levels to the launched sweeps (no tiles, and single
levels of more than 1024 nodes out of the one-work-group sweeps); it is read
once per call, and a captured coarse cycle belongs to one setting.  The routes
share their per-node arithmetic, so the iterates are those of a grid on which it
never changes, bit for bit.
"""
import numpy as np
import pytest

import paper_2606_04292_amd as rsl
from tests.test_gpu_parity import np_
from tests.test_gpu_tile_cycle import CASES
from tests.test_gpu_wg_cycle import N, SINK, VG, _box

pytestmark = pytest.mark.gpu

GRIDS = {"129x65": CASES["129x65_nu2"], "4097": CASES["4097"],
         "33x33": _box([33, 33], VG, [N] * 4, [0.0] * 4),
         "65x257_sink": _box([65, 257], SINK, [N] * 4, [0.0] * 4)}


@pytest.mark.parametrize("precision", [rsl.RS_FP64, rsl.RS_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name", sorted(GRIDS))
def test_switching_between_calls_changes_no_bit(name, precision, monkeypatch):
    def run(modes):
        G = rsl.Grid(GRIDS[name], precision=precision)
        G.begin_step()
        for m in modes:
            if m:
                monkeypatch.setenv("RS_SWEEP", "single")
            else:
                monkeypatch.delenv("RS_SWEEP", raising=False)
            G.sweep(3)
            if precision == rsl.RS_FP64:
                G.vcycle()
            else:
                G.correction_cycle(2)
        x = np_(G.psi())
        G.close()
        return x

    a = run([0, 0, 0, 0])
    assert np.array_equal(a, run([0, 1, 0, 1]))
    assert np.array_equal(a, run([1, 0, 0, 1]))
