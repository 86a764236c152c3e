"""Which form of the step runs where (host only)."""
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


BOX = r"""
#include <cstdio>
#include "lb_internal.h"
int main()
{
    lbk::KParams k{};
    k.nx = k.ny = k.nz = 8;
    k.nsites = 512;
    k.force = 1;
    k.omega_f = k.omega_g = 1.0;
    lbk::set_layout(k, 0, 0);
    const lbk::TileCfg tc = lbk::tile_config(k, 0, false);
    printf("%d %d\n", lbk::step_variant(k, tc, false, 0, false) == lbk::kStepBox,
           lbk::launch_force_collide(k, tc, false, lbk::kStepBox, 0, nullptr, nullptr, nullptr,
                                     nullptr, nullptr) == hipErrorInvalidValue);
}
"""


def test_force_coupling_in_fp64_has_no_box_form(tmp_path):
    """No lattice is sent there, and a launch of it is refused (its kernel is
    FP32 storage's) before anything runs."""
    assert _plan.run(tmp_path, BOX).split() == ["0", "1"]
