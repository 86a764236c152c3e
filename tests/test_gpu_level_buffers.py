"""What the two level buffers hold between calls, also where the steps of one
call hand each other compact levels."""
from __future__ import annotations

import pytest
import torch

import lbinputs
from _gpu import make_lb

pytestmark = pytest.mark.gpu


def _values(lb):
    return [t for t in lb.export_dist() + lb.moments() if t is not None]


# compact g, one site per thread; f's moments too, marching (stress, both
# couplings)
@pytest.mark.parametrize("shape", [(40, 40, 40), (80, 76, 75), (101, 97, 120)])
@pytest.mark.parametrize("coupling,prec", [("stress", "fp64"), ("force", "fp64"),
                                           ("force", "fp32_dev")])
def test_sibling_starts_at_the_level_in_the_first_buffer(shape, coupling, prec):
    """A sibling starts at time level 0 of the shared buffers: the current level
    after an even number of steps, the one a step before it after an odd one."""
    phi0 = lbinputs.spinodal_phi0(shape, seed=29, amp=0.3)
    ref = make_lb(shape, precision=prec, coupling=coupling)
    ref.init_phi(phi0)
    want = []
    for _ in range(7):
        want.append(_values(ref))
        ref.step(1)
    want.append(_values(ref))
    n = float(ref.nsites)
    for calls in ((2,), (3,), (5,), (1, 3), (1, 4), (2, 5), (4, 3)):
        print(f"[sibling] {shape} {coupling} {prec} {calls}", flush=True)
        for sums in (False, True):
            lb = make_lb(shape, precision=prec, coupling=coupling)
            lb.init_phi(phi0)
            rows = []
            for k in calls:
                if sums:
                    rows.append(lb.step_sums(k))
                else:
                    lb.step(k)
            t = sum(calls)
            for a, b in zip(_values(lb), want[t]):
                assert torch.equal(a, b)
            for a, b in zip(_values(lb.sibling("fused")), want[t - t % 2]):
                assert torch.equal(a, b)
            if sums:
                # sums of n terms of order 1 in two orders: n eps of their scale n
                got = torch.cat(rows)[:, 0]
                rho = torch.stack([w[-3].sum() for w in want[:t]])
                assert bool(((got - rho).abs() <= n * n * 2.3e-16).all())


@pytest.mark.parametrize("shape", [(40, 40, 40), (80, 76, 75)])
@pytest.mark.parametrize("coupling,prec", [("stress", "fp64"), ("force", "fp64"),
                                           ("force", "fp32_dev")])
def test_an_earlier_sibling_finds_a_level_in_the_first_buffer(shape, coupling, prec):
    """With a sibling made before, every later call of either context leaves a
    level in the first buffer."""
    phi0 = lbinputs.spinodal_phi0(shape, seed=31, amp=0.3)
    ref = make_lb(shape, precision=prec, coupling=coupling)
    ref.init_phi(phi0)
    want = []
    for _ in range(9):
        want.append(_values(ref))
        ref.step(1)
    lb = make_lb(shape, precision=prec, coupling=coupling)
    lb.init_phi(phi0)
    sib = lb.sibling("fused")
    t = 0
    for k in (3, 2, 3):
        print(f"[sibling] {shape} {coupling} {prec} step {t} + {k}", flush=True)
        lb.step(k)
        t += k
        for a, b in zip(_values(sib), want[t - t % 2]):
            assert torch.equal(a, b)
        for a, b in zip(_values(lb), want[t]):
            assert torch.equal(a, b)
    # and so do the sibling's own steps, from that state (ref is one step on)
    sib.step(3)
    ref.step(1)
    for a, b in zip(_values(lb.sibling("fused")), _values(ref)):
        assert torch.equal(a, b)
