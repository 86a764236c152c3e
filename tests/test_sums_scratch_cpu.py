"""The sums' scratch buffer holds the partials of the steps that run, over the
whole range of lattices (host arithmetic; nothing is launched)."""
from __future__ import annotations

import ctypes
import random
import re

import numpy as np
import pytest

from test_abi_cpu import _params, abi  # noqa: F401  (fixture)

# lattices on which the march takes flat tiles in more workgroups than row tiles
FLAT = [(355, 544, 241), (365, 560, 235), (547, 581, 230), (801, 643, 204), (45, 7821, 121),
        (352, 3733, 54), (301, 575, 228), (53, 7057, 150)]


def _random_shapes(n, seed):
    """Ragged and elongated lattices up to the largest the library takes."""
    rng = random.Random(seed)
    out = []
    while len(out) < n:
        nz = rng.choice([rng.randint(1, 260), rng.randint(1, 1000)])
        ny = int(10 ** rng.uniform(0, 4))
        sites = 10 ** rng.uniform(4, 8.04)
        nx = max(1, int(sites / (ny * nz)))
        if nx * ny * nz < 1.0e8 and ny * nz * 19 * 8 < 2 ** 32:
            out.append((nx, ny, nz))
    return out


def _create(abi, shape, **kw):  # noqa: F811
    """A context over buffers that are never dereferenced, and its scratch in
    partial blocks of 5 FP64."""
    p = _params(abi, nx=shape[0], ny=shape[1], nz=shape[2], **kw)
    s = abi.LbSizes()
    assert abi.lib().lb_query_sizes(ctypes.byref(p), ctypes.byref(s)) == abi.LB_OK
    b = abi.LbBuffers()
    b.state[0], b.state[1], b.phi, b.scratch = 0x1000, 0x2000, 0x3000, 0x4000
    ctx = ctypes.c_void_p()
    assert abi.lib().lb_create(ctypes.byref(p), ctypes.byref(b), None, ctypes.byref(ctx)) == abi.LB_OK
    return ctx, s.scratch_bytes // 40


def _noalloc_blocks(abi, ctx):  # noqa: F811
    """The partial blocks that lb_step_sums_noalloc refuses this context for, or
    0 if the library's array holds them (a call of no steps: no launch)."""
    st = abi.lib().lb_step_sums_noalloc(ctx, 0, ctypes.c_void_p(0x8000))
    m = re.search(rb"over (\d+) partial", abi.lib().lb_last_error()) if st == abi.LB_EINVAL else None
    return int(m.group(1)) if m else 0


@pytest.mark.parametrize("kw", [dict(), dict(tau_g=1.3), dict(halo_x=1), dict(coupling=1),
                                dict(order_param=1), dict(order_param=1, coupling=1),
                                dict(kernel=1), dict(kernel=2), dict(segment_x=3)],
                         ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()) or "default")
@pytest.mark.parametrize("prec", [0, 1])
def test_scratch_holds_the_partials_of_every_step(abi, prec, kw):  # noqa: F811
    for shape in FLAT + _random_shapes(400, seed=5):
        if "halo_x" in kw and shape[0] < 2:
            continue
        ctx, rows = _create(abi, shape, precision=prec, **kw)
        need = _noalloc_blocks(abi, ctx)
        abi.lib().lb_destroy(ctx)
        assert rows >= need, (shape, rows, need)


def _row_blocks(shape, prec, segment_x):
    """Workgroups of the march over row tiles: 8 x 64 or 4 x 128 columns (FP32
    storage with rows of 256 sites: 2 x 256), in segments of segment_x planes
    or the fewest with the least rounds * (planes + 2)."""
    nx, ny, nz = shape
    tz = 64 if 64 * -(-nz // 64) < 128 * -(-nz // 128) else 128
    if prec == 1 and nz == 256:
        tz = 256
    tiles = -(-ny // (512 // tz)) * -(-nz // tz)
    if segment_x:
        return tiles * -(-nx // min(segment_x, nx))
    s = -(-nx // np.arange(1, nx + 1, dtype=np.int64))
    blocks = tiles * -(-nx // s)
    cost = -(-blocks // 256) * (s + 2)
    return int(blocks[int(np.argmin(cost))])


@pytest.mark.parametrize("kw", [dict(), dict(tau_g=1.3), dict(kernel=2), dict(segment_x=2),
                                dict(segment_x=5, halo_x=1)],
                         ids=["default", "tau_g1.3", "stream", "segment2", "segment5-shard"])
@pytest.mark.parametrize("prec", [0, 1])
def test_noalloc_sums_take_every_lattice_whose_row_tiles_fit(abi, prec, kw):  # noqa: F811
    """Whatever tiling the march runs over."""
    fits = 0
    pairs = [(4182, 1, 256), (1106, 13, 256), (10606, 1, 256), (2, 8191, 256)]
    for shape in FLAT + pairs + _random_shapes(400, seed=6):
        if "halo_x" in kw and shape[0] < 2:
            continue
        ctx, _ = _create(abi, shape, precision=prec, **kw)
        need = _noalloc_blocks(abi, ctx)
        abi.lib().lb_destroy(ctx)
        blocks = _row_blocks(shape, prec, kw.get("segment_x", 0))
        fit = blocks <= abi.NOALLOC_MAX_PARTIALS
        fits += fit
        assert (need == 0) == fit, (shape, need, blocks)
    assert fits > 150
