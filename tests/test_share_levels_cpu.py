"""Argument checks of lb_share_levels, before any HIP call."""
from __future__ import annotations

import ctypes

from test_abi_cpu import _params, abi  # noqa: F401  (fixture)


def test_share_levels_of_a_fresh_context_needs_no_buffer(abi):  # noqa: F811
    L = abi.lib()
    ctx = ctypes.c_void_p()
    b = abi.LbBuffers()
    b.state[0], b.state[1], b.phi, b.scratch = 0x1000, 0x2000, 0x3000, 0x4000
    p = _params(abi)
    assert L.lb_create(ctypes.byref(p), ctypes.byref(b), None, ctypes.byref(ctx)) == abi.LB_OK
    assert L.lb_share_levels(None, None) == abi.LB_EINVAL
    assert L.lb_share_levels(ctx, None) == abi.LB_OK
    L.lb_destroy(ctx)
