"""Argument checks of the calls that take many levels, before any HIP call."""
from __future__ import annotations

import ctypes

import pytest

from test_abi_cpu import _params, abi  # noqa: F401  (fixture)


def _arr(*p):
    return (ctypes.c_void_p * len(p))(*p)


@pytest.mark.parametrize("order_param", [0, 1])
def test_chains_validate_without_launching(abi, order_param):  # noqa: F811
    L = abi.lib()
    ctx = ctypes.c_void_p()
    b = abi.LbBuffers()
    b.state[0], b.state[1], b.phi, b.scratch = 0x1000, 0x2000, 0x3000, 0x4000
    p = _params(abi, order_param=order_param)
    assert L.lb_create(ctypes.byref(p), ctypes.byref(b), None, ctypes.byref(ctx)) == abi.LB_OK
    try:
        src = ctypes.c_void_p(0x10000)
        two = _arr(0x20000, 0x30000)
        assert L.lb_step_chain(None, src, two, None, 2) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, None, two, None, 2) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, two, None, -1) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, None, None, 2) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, _arr(0x20000, None), None, 2) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, _arr(0x10000), None, 1) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, _arr(0x20000, 0x20000), None, 2) == abi.LB_EINVAL
        assert L.lb_step_chain(ctx, src, _arr(0x20000, 0x30010), None, 2) == abi.LB_EALIGN
        assert L.lb_step_chain(ctx, ctypes.c_void_p(0x10010), two, None, 2) == abi.LB_EALIGN
        phis = _arr(None, 0x40010)
        assert L.lb_step_chain(ctx, src, two, phis, 2) == (abi.LB_EINVAL if order_param
                                                           else abi.LB_EALIGN)
        assert L.lb_step_chain(ctx, src, None, None, 0) == abi.LB_OK
        assert L.lb_level_phi(ctx, None, src) == abi.LB_EINVAL
        assert L.lb_level_phi(ctx, src, None) == abi.LB_EINVAL
        assert L.lb_level_phi(ctx, src, ctypes.c_void_p(0x50010)) == abi.LB_EALIGN
        assert L.lb_adjoint_chain(None, two, None, 2, None) == abi.LB_EINVAL
        assert L.lb_adjoint_chain(ctx, None, None, 2, None) == abi.LB_EINVAL
        assert L.lb_adjoint_chain(ctx, two, None, -1, None) == abi.LB_EINVAL
        assert L.lb_adjoint_chain(ctx, _arr(0x20000, None), None, 2, None) == abi.LB_EINVAL
        assert L.lb_adjoint_chain(ctx, _arr(0x20010), None, 1, None) == abi.LB_EALIGN
        # no adjoint buffers
        assert L.lb_adjoint_chain(ctx, two, None, 2, None) == abi.LB_ESTATE
    finally:
        L.lb_destroy(ctx)


@pytest.mark.parametrize("last_state", [0, 1])
def test_segment_validates_as_the_chain(abi, last_state):  # noqa: F811
    L = abi.lib()
    ctx = ctypes.c_void_p()
    b = abi.LbBuffers()
    b.state[0], b.state[1], b.phi, b.scratch = 0x1000, 0x2000, 0x3000, 0x4000
    p = _params(abi)
    assert L.lb_create(ctypes.byref(p), ctypes.byref(b), None, ctypes.byref(ctx)) == abi.LB_OK
    try:
        src = ctypes.c_void_p(0x10000)
        two = _arr(0x20000, 0x30000)
        assert L.lb_step_segment(None, src, two, None, 2, last_state) == abi.LB_EINVAL
        assert L.lb_step_segment(ctx, src, _arr(0x20000, 0x20000), None, 2,
                                 last_state) == abi.LB_EINVAL
        assert L.lb_step_segment(ctx, src, two, _arr(None, 0x40010), 2, last_state) == abi.LB_EALIGN
        assert L.lb_step_segment(ctx, src, two, _arr(0x40000, 0x40000), 2,
                                 last_state) == abi.LB_EINVAL
        assert L.lb_step_segment(ctx, src, None, None, 0, last_state) == abi.LB_OK
    finally:
        L.lb_destroy(ctx)
