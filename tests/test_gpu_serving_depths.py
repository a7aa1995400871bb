"""The serving engine's levels between the wide ones and the one-work-group cycle.

A level that is small enough for one work-group but does not fit its LDS cycle
(65^2, 17^3, a 4097-node column) runs as a wide one while the engine has a
depth left, else from memory inside the small-level kernel: max_wide_levels
sends requests there.  Results against the oracle's converged steps (1e-10),
with and without graphs, and the same bits whether a request runs alone or in
a mix whose depth changes while it runs.
"""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2606_04292_amd as rsl
from paper_2606_04292_amd import serve
from tests.test_gpu_parity import rel, say
from tests.test_gpu_serving import TOL_CONV, oracle_solution, serve_all
from tests.test_gpu_wg_cycle import D, F, HK, N, VG, _box

pytestmark = pytest.mark.gpu

REQUESTS = {
    "65x65": _box([65, 65], VG, [N, N, F, N], [0.0] * 4, patch=(3, (20, 0), (44, 0))),
    "17x17x17": _box([17, 17, 17], HK, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
    "5x5x65": _box([5, 5, 65], VG, [N] * 4 + [D, N], [0.0] * 4 + [-1.0, 0.0]),
    # one level only, sweeps without a coarser grid: 106 corrections in a step
    "3x2049": _box([3, 2049], VG, [N, N, D, D], [0, 0, -0.8, -0.5]),
    "4097": _box([4097], VG, [F, N], [0.0, 0.0]),
    "129x129": _box([129, 129], VG, [N, D, N, N], [0.0, -0.7, 0.0, 0.0]),
    "33x33": _box([33, 33], VG, [N, N, D, N], [0, 0, -0.8, 0.0]),
}


@pytest.fixture(scope="module")
def reference():
    return {k: oracle_solution(w) for k, w in REQUESTS.items()}


def _check(names, res, reference):
    for q, k in enumerate(names):
        psi, st = res[q]
        assert st.state == serve.RS_REQ_FINISHED and st.status == rsl.RS_OK, k
        e = rel(psi, reference[k])
        say("  request", k, "corrections", st.corrections, "rel", e)
        assert e <= TOL_CONV, k


# levels above 8192 nodes need a depth: 129x129 is served from one wide level on
@pytest.mark.parametrize("graph", [1, 0])
@pytest.mark.parametrize("wide", [0, 1, 4])
def test_small_levels_from_memory_match_the_oracle(wide, graph, reference):
    names = [k for k in REQUESTS if wide > 0 or k != "129x129"]
    say("max_wide_levels", wide, "graph", graph)
    res = serve_all([REQUESTS[k] for k in names],
                    serve.engine_opts(max_wide_levels=wide, tail_nodes=8192, use_graph=graph,
                                      max_corrections=2000))
    _check(names, res, reference)


def test_results_do_not_depend_on_the_depths_in_the_mix(reference):
    """Requests of no, one and several wide levels join one after the other: each depth's
    round is run, and every result has the bits it has alone."""
    names = ["33x33", "65x65", "129x129", "17x17x17", "4097"]
    opts = serve.engine_opts(max_wide_levels=4, tail_nodes=300, use_graph=1, rounds_per_tick=1)
    mix = serve_all([REQUESTS[k] for k in names], opts, schedule=[0, 2, 4, 5, 30])
    _check(names, mix, reference)
    for q, k in enumerate(names):
        alone = serve_all([REQUESTS[k]], opts)[0][0]
        assert np.array_equal(alone, mix[q][0]), k
