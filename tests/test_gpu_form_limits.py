"""The form that a step takes by its size against the two passes, bit for bit,
on lattices on either side of where FP32 storage marches again."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import lbinputs
from _gpu import make_lb

pytestmark = pytest.mark.gpu

# the LB scheme: one plane per segment up to 90000 sites (the first two), two
# planes or more sites (the others); finite differences: two planes per segment
# from 200000 to 270000 sites (the first four), fewer sites or more planes or
# sites
LB = [(42, 42, 44), (44, 40, 50), (30, 35, 75), (44, 44, 44), (36, 56, 50)]
FD = [(64, 50, 64), (50, 64, 64), (60, 60, 60), (64, 64, 64), (56, 56, 56), (52, 60, 70),
      (22, 100, 128)]


@pytest.mark.parametrize("order_param,shape", [("lb", s) for s in LB] + [("fd", s) for s in FD])
@pytest.mark.parametrize("tau_g", [1.0, 1.3])
def test_default_form_and_two_passes_agree_bit_for_bit(shape, order_param, tau_g):
    print(f"[limits] {shape} {order_param} tau_g {tau_g}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=47, amp=0.3)
    states, sums = [], []
    for kernel in ("fused", "two_pass"):
        lb = make_lb(shape, precision="fp32_dev", tau_f=0.8, tau_g=tau_g, order_param=order_param,
                     kernel=kernel)
        lb.init_phi(phi0)
        lb.step(2)
        sums.append(lb.step_sums(3).cpu().numpy())
        states.append([t for t in lb.export_dist() + lb.moments() if t is not None])
    for a, b in zip(*states):
        assert torch.equal(a, b)
    # five sums of n terms of order 1 in two orders: n eps of their scale n
    n = float(np.prod(shape))
    assert np.abs(sums[0] - sums[1]).max() <= n * n * 2.3e-16
