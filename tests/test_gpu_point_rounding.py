"""Rounding of the FP64 pointwise solve.

A medium that hardly conducts has one equation per node, a theta(psi) = g.
Swept to rounding, the error of psi against that equation in extended
precision (64-bit mantissas) is that of the terms' own roundings, a few
half-ulps of psi (more where theta is flat), and no shift common to the whole
grid.  A factor of a theta that is rounded once for every node shifts all of
them one way: with a = 3/(2 30 s) and theta_s - theta_r = 0.38 its rounding
error is 0.8 of the largest there can be, and moved the mean by 2 half-ulps.

Tolerance for the mean, in half-ulps of psi: 0.5 for the law functions' own
mean error and four standard deviations, 4 * 3.5 / sqrt(N), of the mean of N
independent roundings.
"""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2606_04292_amd as rsl
from paper_2606_04292_amd import workloads as W
from tests.test_gpu_parity import np_, say
from tests.test_gpu_wg_cycle import HK, N, VG, _box

pytestmark = pytest.mark.gpu

X = np.longdouble


def _theta(law, psi):
    """theta - theta_r and theta' in extended precision (psi < 0)."""
    d = X(law.theta_s) - X(law.theta_r)
    if law.model == W.MODEL_HAVERKAMP:
        hu = -X(law.psi_unit) * psi
        Q = hu ** X(law.hk_beta)
        th = d * X(law.hk_alpha) / (X(law.hk_alpha) + Q)
        return th, X(law.psi_unit) * X(law.hk_beta) * th * Q / (hu * (X(law.hk_alpha) + Q))
    m = X(1.0 - 1.0 / law.vg_n)   # the double that the solver holds
    P = (-X(law.vg_alpha) * psi) ** X(law.vg_n)
    Se = (1 + P) ** -m
    return d * Se, d * m * X(law.vg_n) * P * Se / ((1 + P) * -psi)


# one work-group, and one launch per colour
@pytest.mark.parametrize("n", [[2049], [129, 65]], ids=["2049", "129x65"])
@pytest.mark.parametrize("model", ["vgm", "haverkamp"])
def test_pointwise_fixed_point_has_no_common_shift(model, n):
    law = dataclasses.replace(VG if model == "vgm" else HK, theta_s=0.43, theta_r=0.05, Ks=1e-40,
                              xi=0.0, kappa_rule=W.KAPPA_CONST, kappa=0.0, newton_iters=30,
                              newton_tol=0.0)
    w = dataclasses.replace(_box(n, law, [N] * (2 * len(n)), [0.0] * (2 * len(n))), dt=30.0)
    G = rsl.Grid(w)
    psi = torch.as_tensor(w.psi0, device=G.device)
    G.set_state(psi, psi * 1.01, nstep=1)
    G.begin_step(order=2)
    G.sweep(3)
    x, g = np_(G.psi()), np_(G.field(rsl.FIELD_G))
    G.close()
    a = X(1.5 / 30.0)
    th, dth = _theta(law, x.astype(X))
    e = (a * (X(law.theta_r) + th) - g.astype(X)) / (a * dth)
    e = (e / (0.5 * np.spacing(np.abs(x)))).astype(np.float64)
    mean, rms = e.mean(), np.sqrt(np.mean(e * e))
    say("fixed point", model, n, "error in half-ulps of psi: mean %.3f, rms %.3f" % (mean, rms))
    assert abs(mean) <= 0.5 + 4 * 3.5 / np.sqrt(e.size)
