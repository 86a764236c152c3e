"""What the host layer plans for a lattice, from the built library: a small
program against its internal header, for tests that check which form of the
step a size takes.  Host arithmetic; nothing is launched."""
from __future__ import annotations

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1609_01479_amd")

SOURCE = r"""
#include <cstdio>
#include "lb_internal.h"
int main()
{
    int nx, ny, nz, seg, fp32;
    double tau_g;
    while (scanf("%d %d %d %d %d %lf", &nx, &ny, &nz, &seg, &fp32, &tau_g) == 6) {
        lbk::KParams k{};
        k.nx = nx;
        k.ny = ny;
        k.nz = nz;
        k.nsites = nx * ny * nz;
        k.omega_f = 1.0;
        k.omega_g = 1.0 / tau_g;
        lbk::set_layout(k, 0, 0);
        const lbk::TileCfg tc = lbk::tile_config(k, seg, fp32);
        printf("%d %d %d\n", tc.tz, tc.ntiles, tc.nseg);
    }
}
"""


def run(tmp_path, source, text=""):
    """What a program against the library's internal header prints."""
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), str(src),
                    "-o", str(exe), os.path.join(PKG, "liblbmi.so"), f"-Wl,-rpath,{PKG}",
                    "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout


def tilings(tmp_path, lattices):
    """(tile width, tiles, segments) of the march of the LB scheme's step for
    each (shape, segment_x, FP32 storage, tau_g); width 0: flat tiles."""
    text = "".join(f"{x} {y} {z} {seg} {int(fp32)} {tau_g}\n"
                   for (x, y, z), seg, fp32, tau_g in lattices)
    return [tuple(map(int, line.split())) for line in run(tmp_path, SOURCE, text).splitlines()]
