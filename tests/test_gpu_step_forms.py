"""The forms of the LB step: the marching kernel (flat and row tiles) and the
two passes give the same levels bit for bit, at the edges of their ranges."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import lbinputs
import oracle
from _gpu import field_errors, gpu_state, make_lb, oracle_params, oracle_state

pytestmark = pytest.mark.gpu

# (shape, segment_x): planes of exactly one flat tile, one site and one row
# more (last tile shifted back), rows longer than any halo allows (row tiles),
# the longest flat rows of each precision, whole-row tiles, rows of 1 and 2
# sites, extents of 1 and 2, tiles that start and end anywhere in a row
MARCH = [((8, 8, 64), 8), ((9, 27, 19), 8), ((2, 9, 64), 1), ((8, 3, 254), 8), ((8, 3, 255), 8),
         ((9, 5, 256), 9), ((2, 3, 257), 1), ((8, 513, 1), 8), ((8, 300, 2), 8), ((9, 11, 100), 8),
         ((8, 13, 150), 8), ((8, 7, 74), 8), ((8, 2, 256), 8), ((9, 6, 96), 9), ((3, 5, 100), 2)]


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("shape,seg", MARCH)
def test_march_and_two_passes_agree_bit_for_bit(shape, seg, prec, tau_g):
    print(f"[forms] {shape} seg {seg} {prec} tau_g {tau_g}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=31, amp=0.3)
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


@pytest.mark.parametrize("coupling", ["stress", "force"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (4, 4, 4), (5, 13, 1), (32, 32, 64), (29, 37, 61),
                                   (64, 64, 64)])
def test_default_step_sums_rows_are_the_levels_sums(shape, prec, coupling):
    """Blocks of one wave and of four (up to and beyond 65536 sites), and the
    sums of several steps reduced by one launch: every row is lb_sums of its
    level, over more steps than one launch holds for the larger lattices."""
    print(f"[sums] {shape} {prec} {coupling}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=7, amp=0.3)
    lb = make_lb(shape, precision=prec, tau_f=0.8, coupling=coupling)
    ref = make_lb(shape, precision=prec, tau_f=0.8, coupling=coupling)
    lb.init_phi(phi0)
    ref.init_phi(phi0)
    rows = lb.step_sums(6).cpu().numpy()
    n = float(np.prod(shape))
    for t in range(6):
        assert np.abs(rows[t] - ref.sums().cpu().numpy()).max() <= n * n * 2.3e-16
        ref.step(1)
    for a, b in zip(gpu_state(lb), gpu_state(ref)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("shape,seg", [((5, 11, 100), 4), ((2, 9, 64), 1), ((3, 3, 257), 3),
                                       ((9, 6, 11), 0)])
def test_fp64_forms_match_the_oracle(shape, seg, tau_g):
    phi0 = lbinputs.spinodal_phi0(shape, seed=12, amp=0.3)
    lb = make_lb(shape, tau_f=0.8, tau_g=tau_g, segment_x=seg)
    lb.init_phi(phi0)
    lb.step(5)
    p = oracle_params(shape, tau_f=0.8, tau_g=tau_g)
    f, g = oracle.run(p, *oracle.init(p, phi0), 5)
    errs = field_errors(gpu_state(lb), oracle_state(p, f, g))
    assert max(errs.values()) <= 1e-12, errs


@pytest.mark.parametrize("layout", [dict(layout="soa"), dict(layout="aos"),
                                    dict(layout="aosoa", aosoa_len=4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
def test_flat_tiles_in_every_layout(prec, layout):
    shape = (9, 9, 100)
    phi0 = lbinputs.spinodal_phi0(shape, seed=3, amp=0.3)
    out = []
    for lay in ({}, layout):
        lb = make_lb(shape, precision=prec, tau_f=0.8, tau_g=1.3, segment_x=8, **lay)
        lb.init_phi(phi0)
        lb.step(4)
        out.append(gpu_state(lb))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_noalloc_still_refuses_what_row_tiles_exceed():
    """The allocation-free sums' limit is stated for the march over row tiles,
    whichever form runs."""
    from paper_1609_01479_amd._abi import LbError
    out = torch.empty((1, 5), dtype=torch.float64, device="cuda:0")
    for kw in (dict(), dict(coupling="force")):
        with pytest.raises(LbError, match="partial blocks"):
            make_lb((1, 60000, 1), **kw).step_sums_noalloc(1, out)


@pytest.mark.parametrize("coupling,order_param", [("force", "lb"), ("stress", "fd"), ("force", "fd")])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("shape,seg", [((1, 1, 1), 1), ((5, 9, 70), 3), ((4, 6, 64), 4),
                                       ((33, 40, 50), 7), ((3, 5, 131), 2), ((116, 116, 116), 0)])
def test_other_schemes_forms_agree_bit_for_bit(shape, seg, prec, coupling, order_param):
    """March and two passes of the other schemes: blocks of one wave and of
    four, rows that are whole 64-byte pieces and rows that are not, and (at
    116^3) the update pass that marches."""
    print(f"[forms] {shape} seg {seg} {prec} {coupling} {order_param}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=31, amp=0.3)
    states, sums = [], []
    for kernel, sx in (("fused", seg), ("two_pass", 0)):
        lb = make_lb(shape, precision=prec, tau_f=0.8, coupling=coupling, order_param=order_param,
                     kernel=kernel, segment_x=sx)
        lb.init_phi(phi0)
        lb.step(2)
        sums.append(lb.step_sums(3).cpu().numpy())
        states.append([t for t in lb.export_dist() + lb.moments() if t is not None])
    for a, b in zip(*states):
        assert torch.equal(a, b)
    n = float(np.prod(shape))
    assert np.abs(sums[0] - sums[1]).max() <= n * n * 2.3e-16


@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("yz", [(1, 1), (5, 9), (128, 128), (129, 128)])
def test_faces_packed_together_and_one_at_a_time_agree(yz, prec):
    """Faces below and beyond the size that deals slots to more threads; either
    buffer may be missing, and then its side is left alone."""
    shape = (4,) + yz
    print(f"[faces] {shape} {prec}", flush=True)
    phi0 = lbinputs.spinodal_phi0((shape[0] + 2,) + yz, seed=5, amp=0.3)
    lb = make_lb(shape, precision=prec, halo_x=True)
    lb.init_phi(phi0)
    lb.step(1)
    both = [lb.new_face().zero_(), lb.new_face().zero_()]
    single = [lb.new_face().zero_(), lb.new_face().zero_()]
    lb.pack_faces(*both)
    lb.pack_faces(single[0], None)
    lb.pack_faces(None, single[1])
    assert torch.equal(both[0], single[0]) and torch.equal(both[1], single[1])
    assert both[0].any() and both[1].any()
    start = lb.get_state()
    lb.unpack_faces(both[1], both[0])
    want = lb.get_state()
    lb.set_state(start)
    lb.unpack_faces(both[1], None)
    lb.unpack_faces(None, both[0])
    assert torch.equal(lb.get_state(), want)


@pytest.mark.parametrize("order_param", ["lb", "fd"])
@pytest.mark.parametrize("coupling", ["stress", "force"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 2, 7), (32, 32, 64), (41, 40, 40), (65, 64, 64)])
def test_moments_alone_and_together_agree(shape, prec, coupling, order_param):
    """lb_moments of any subset of its outputs gives the same values, phi alone
    included (a pass of its own), and lb_sums is their sum: blocks of one wave
    and of four, and more blocks than the sums' partials."""
    print(f"[moments] {shape} {prec} {coupling} {order_param}", flush=True)
    lb = make_lb(shape, precision=prec, tau_f=0.8, coupling=coupling, order_param=order_param)
    lb.init_phi(lbinputs.spinodal_phi0(shape, seed=17, amp=0.3))
    lb.step(3)
    rho, u, phi = lb.moments()
    for want in ((1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (0, 1, 1), (1, 0, 1)):
        got = [torch.full_like(v, 7.0) for v in (rho, u, phi)]
        lb._call("lb_moments", *(v.data_ptr() if w else None for v, w in zip(got, want)))
        for v, g, w in zip((rho, u, phi), got, want):
            assert torch.equal(g, v if w else torch.full_like(v, 7.0))
    s = lb.sums()
    ref = torch.stack([rho.sum(), phi.sum(), *((rho * u[k]).sum() for k in range(3))])
    # two orders of n FP64 terms: 2 n eps of the sum of their sizes, and one
    # rounding each for the division by rho and the product with it
    n = float(np.prod(shape))
    size = torch.stack([rho.sum(), phi.abs().sum(), *((rho * u[k]).abs().sum() for k in range(3))])
    assert bool(((s - ref).abs() <= (2.0 * n + 4.0) * 2.3e-16 * size).all())


# (shape): below and above the sites from which a call's steps hand each other
# compact levels (40000), and from which their phi pass marches (FP64 160000,
# with the force 200000, FP32 storage 650000): extents that its 12 x 32 tile
# divides, covers once, shifts back or is larger than, thin slabs, few and many
# planes, more sites than the sums have workgroups for; and from which the
# levels hold f's moments with tau_f = 1 (FP64 450000, with the force 800000,
# FP32 storage 1500000)
COMPACT = [(33, 33, 36), (40, 25, 40), (34, 11, 107), (70, 48, 64), (4, 203, 257), (57, 61, 63),
           (3, 200, 300), (41, 5, 1000), (9000, 11, 7), (88, 90, 83), (101, 97, 120),
           (4, 352, 360), (75, 84, 96), (37, 203, 214)]


@pytest.mark.parametrize("tau_f", [1.0, 0.8])
@pytest.mark.parametrize("coupling,prec", [("stress", "fp64"), ("force", "fp64"),
                                           ("force", "fp32_dev")])
@pytest.mark.parametrize("shape", COMPACT)
def test_steps_of_one_call_are_those_of_many(shape, coupling, prec, tau_f):
    """Steps of one call hand each other compact levels (tau_g = 1); one step
    per call makes full ones: the same levels bit for bit."""
    print(f"[compact] {shape} {coupling} {prec} tau_f {tau_f}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=23, amp=0.3)
    one = make_lb(shape, precision=prec, tau_f=tau_f, coupling=coupling)
    many = make_lb(shape, precision=prec, tau_f=tau_f, coupling=coupling)
    one.init_phi(phi0)
    many.init_phi(phi0)
    sums = []
    for _ in range(7):
        sums.append(many.sums().cpu().numpy())
        many.step(1)
    one.step(2)
    rows = one.step_sums(3).cpu().numpy()
    one.step(2)
    for a, b in zip(gpu_state(one), gpu_state(many)):
        assert np.array_equal(a, b)
    # five sums of n terms of order 1 in two orders: n eps of their scale n
    n = float(np.prod(shape))
    for t in range(3):
        assert np.abs(rows[t] - sums[2 + t]).max() <= n * n * 2.3e-16


@pytest.mark.parametrize("coupling,prec", [("stress", "fp64"), ("force", "fp64"),
                                           ("force", "fp32_dev")])
@pytest.mark.parametrize("shape", [(34, 36, 40), (70, 48, 64)])
def test_rollout_through_compact_levels(shape, coupling, prec):
    """A rollout hands its levels on compact within a segment; with a
    checkpoint at every step each segment is one step and every level full.
    The same phi and gradients bit for bit."""
    from paper_1609_01479_amd.rollout import rollout
    print(f"[compact rollout] {shape} {coupling} {prec}", flush=True)
    got = []
    for interval in (1, 3, 7):
        phi0 = torch.tensor(lbinputs.spinodal_phi0(shape, seed=5, amp=0.3), device="cuda:0",
                            requires_grad=True)
        theta = [torch.tensor(v, dtype=torch.float64, device="cuda:0", requires_grad=True)
                 for v in (-0.00625, 0.00625, 0.004)]
        phi = rollout(phi0, *theta, 7, interval=interval, precision=prec, coupling=coupling,
                      tau_f=0.8)
        grads = torch.autograd.grad((phi ** 2).sum(), [phi0] + theta)
        got.append([phi.detach()] + list(grads))
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)


# one box, boxes shifted back and larger than the lattice, as many boxes as the
# form takes (512, with the force coupling 256) and more
BOX = [(1, 1, 1), (1, 2, 3), (4, 4, 4), (5, 4, 9), (3, 17, 6), (2, 70, 9), (13, 18, 11),
       (32, 32, 16), (33, 32, 16), (32, 32, 32), (33, 32, 32)]


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("coupling,prec", [("stress", "fp64"), ("stress", "fp32_dev"),
                                           ("force", "fp32_dev")])
@pytest.mark.parametrize("shape", BOX)
def test_box_step_and_two_passes_agree_bit_for_bit(shape, coupling, prec, tau_g):
    print(f"[box] {shape} {coupling} {prec} tau_g {tau_g}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=37, amp=0.3)
    states, sums, phis = [], [], []
    for kernel in ("fused", "two_pass"):
        lb = make_lb(shape, precision=prec, tau_f=0.8, tau_g=tau_g, coupling=coupling, kernel=kernel)
        lb.init_phi(phi0)
        lb.step(2)
        sums.append(lb.step_sums(3).cpu().numpy())
        src, dst = lb.get_state(), lb.new_state()
        phis.append(torch.empty(shape, dtype=torch.float64, device="cuda:0"))
        lb.step_chain(src, [dst], [phis[-1]])
        lb.set_state(dst)
        states.append(gpu_state(lb))
    for a, b in zip(*states):
        assert np.array_equal(a, b)
    assert torch.equal(*phis)
    # five sums of n terms of order 1 in two orders: n eps of their scale n
    n = float(np.prod(shape))
    assert np.abs(sums[0] - sums[1]).max() <= max(n, 4.0) * n * 2.3e-16


@pytest.mark.parametrize("tau_g", [1.0, 1.3])
@pytest.mark.parametrize("coupling", ["stress", "force"])
@pytest.mark.parametrize("prec", ["fp64", "fp32_dev"])
@pytest.mark.parametrize("shape", BOX)
def test_fd_box_step_and_two_passes_agree_bit_for_bit(shape, prec, coupling, tau_g):
    print(f"[fd box] {shape} {coupling} {prec} tau_g {tau_g}", flush=True)
    phi0 = lbinputs.spinodal_phi0(shape, seed=41, amp=0.3)
    states, sums = [], []
    for kernel in ("fused", "two_pass"):
        lb = make_lb(shape, precision=prec, tau_f=0.8, tau_g=tau_g, coupling=coupling,
                     order_param="fd", kernel=kernel)
        lb.init_phi(phi0)
        lb.step(2)
        sums.append(lb.step_sums(3).cpu().numpy())
        f, _ = lb.export_dist()
        states.append([f.cpu().numpy(), lb.phi().cpu().numpy()])
    for a, b in zip(*states):
        assert np.array_equal(a, b)
    # five sums of n terms of order 1 in two orders: n eps of their scale n
    n = float(np.prod(shape))
    assert np.abs(sums[0] - sums[1]).max() <= max(n, 4.0) * n * 2.3e-16
