"""The LB step's march over flat tiles (consecutive sites of a plane) against
the two passes, bit for bit, at the edges of what flat tiles take.

Lattices of at most 120000 sites march over row tiles whatever their extents,
so these are just above that; test_tilings_cpu.py holds the library to the
tiling each entry is for."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import lbinputs
import oracle
from _gpu import field_errors, gpu_state, make_lb, oracle_params, oracle_state

pytestmark = pytest.mark.gpu

BOTH, FP32 = ("fp64", "fp32_dev"), ("fp32_dev",)
# (shape, segment_x, precisions that take flat tiles): a plane of exactly one
# tile, of one site and of one row more (the last tile shifted back, its sites
# counted once in the sums), of rows that a tile holds whole (FP32: no diagonal
# cells of their own), the longest rows whose halo fits, rows of 1 and 2 sites,
# tiles that start and end anywhere in a row, several tiles, one segment,
# segments of 1 and 2 planes and a last one cut short
FLAT = [((235, 8, 64), 8, FP32), ((234, 27, 19), 8, BOTH), ((234, 27, 19), 2, BOTH),
        ((209, 9, 64), 8, FP32), ((158, 3, 254), 8, FP32), ((94, 5, 256), 9, FP32),
        ((235, 2, 256), 8, FP32), ((234, 513, 1), 8, BOTH), ((235, 512, 1), 9, BOTH),
        ((201, 300, 2), 8, BOTH), ((235, 256, 2), 8, BOTH),
        ((110, 11, 100), 8, BOTH), ((62, 13, 150), 8, BOTH),
        ((232, 7, 74), 8, BOTH), ((209, 6, 96), 9, BOTH), ((8, 105, 150), 8, BOTH),
        ((228, 16, 33), 9, BOTH), ((86, 7, 200), 300, BOTH),
        ((62, 13, 150), 1, ("fp64",))]


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("shape,seg,prec", [(s, seg, q) for s, seg, p in FLAT for q in p])
def test_flat_march_and_two_passes_agree_bit_for_bit(shape, seg, prec, tau_g):
    print(f"[flat] {shape} seg {seg} {prec} tau_g {tau_g}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=43, amp=0.3)
    states, sums = [], []
    for kernel, sx in (("fused", seg), ("two_pass", 0)):
        lb = make_lb(shape, precision=prec, tau_f=0.8, tau_g=tau_g, kernel=kernel, segment_x=sx)
        lb.init_phi(phi0)
        lb.step(2)
        sums.append(lb.step_sums(3).cpu().numpy())
        states.append(gpu_state(lb))
    for a, b in zip(*states):
        assert np.array_equal(a, b)
    # five sums of n terms of order 1 in two orders: n eps of their scale n
    n = float(np.prod(shape))
    assert np.abs(sums[0] - sums[1]).max() <= n * n * 2.3e-16


@pytest.mark.parametrize("layout", [dict(layout="soa"), dict(layout="aos"),
                                    dict(layout="aosoa", aosoa_len=4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
def test_flat_march_in_every_layout(prec, layout):
    shape = (110, 11, 100)
    phi0 = lbinputs.spinodal_phi0(shape, seed=3, amp=0.3)
    out = []
    for lay in ({}, layout):
        lb = make_lb(shape, precision=prec, tau_f=0.8, tau_g=1.3, segment_x=8, **lay)
        lb.init_phi(phi0)
        lb.step(3)
        out.append(gpu_state(lb))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("shape", [(62, 13, 150), (110, 11, 100)])
def test_fp64_flat_march_matches_the_oracle(shape, tau_g):
    phi0 = lbinputs.spinodal_phi0(shape, seed=12, amp=0.3)
    lb = make_lb(shape, tau_f=0.8, tau_g=tau_g, segment_x=8)
    lb.init_phi(phi0)
    lb.step(5)
    p = oracle_params(shape, tau_f=0.8, tau_g=tau_g)
    f, g = oracle.run(p, *oracle.init(p, phi0), 5)
    errs = field_errors(gpu_state(lb), oracle_state(p, f, g))
    assert max(errs.values()) <= 1e-12, errs


C = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
     (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
     (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]


@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
def test_flat_twin_streams_freely(prec):
    """The march's memory-only twin moves every population one cell along its
    direction (post-propagation values: the step's pull, so f_i(x) comes from
    x - c_i of the level before)."""
    shape = (110, 11, 100)
    lb = make_lb(shape, precision=prec, segment_x=8, tau_f=0.8, tau_g=1.3)
    lb.init_phi(lbinputs.spinodal_phi0(shape, seed=3, amp=0.3))
    lb.step(2)
    f0, _ = lb.export_dist()
    twin = lb.sibling("stream")
    twin.step(1)
    f1, _ = twin.export_dist()
    for i, c in enumerate(C):
        assert torch.equal(f1[i], torch.roll(f0[i], c, (0, 1, 2))), i
