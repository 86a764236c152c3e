"""The lattices of the flat-tile tests march over flat tiles (host only)."""
from __future__ import annotations

import _plan
import test_gpu_flat_tiles as gpu


def test_flat_tile_lattices_take_flat_tiles(tmp_path):
    cases = [(shape, seg, prec, tau_g) for shape, seg, precs in gpu.FLAT
             for prec in precs for tau_g in (1.0, 1.3)]
    cases += [((110, 11, 100), 8, prec, 1.3) for prec in gpu.BOTH]
    cases += [((62, 13, 150), 8, "fp64", 1.3)]
    got = _plan.tilings(tmp_path, [(s, seg, prec == "fp32_dev", tau_g)
                                   for s, seg, prec, tau_g in cases])
    assert len(got) == len(cases)
    for case, (tz, tiles, nseg) in zip(cases, got):
        assert tz == 0, case
        assert tiles == -(-case[0][1] * case[0][2] // 512), case
