"""The FP64 step rounds a collided population once after its even part."""
from __future__ import annotations

import numpy as np
import pytest

from _gpu import make_lb

pytestmark = pytest.mark.gpu

C = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
     (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
     (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
W = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)


@pytest.mark.parametrize("kw", [dict(), dict(kernel="two_pass"), dict(segment_x=4)],
                         ids=["boxes", "two_passes", "march"])
def test_populations_are_rounded_once(kw):
    """tau_f = 1 and phi = 0: f*_i = w (q_i +- 3 c_i.j) with q_i even in c_i.  The
    sum of an opposite pair is 2 w q up to the roundings of the two: 0.41 ulp
    (rms: sqrt 2 times 1/sqrt 12) with w q +- 3 w c.j rounded once each, 0.71
    with w q rounded before (its error comes in twice, if independent of theirs;
    measured 0.58)."""
    shape = (12, 10, 16)
    rng = np.random.default_rng(11)
    f = W[:, None, None, None] * (0.9 + 0.05 * rng.uniform(-1, 1, (19,) + shape))
    lb = make_lb(shape, tau_f=1.0, tau_g=1.0, **kw)
    lb.import_dist(f, np.zeros_like(f))
    lb.step(1)
    out = lb.export_dist()[0].cpu().numpy()
    star = np.stack([np.roll(out[i], [-c for c in C[i]], (0, 1, 2)) for i in range(19)])
    # q as the step forms it: b summed in index order, then one rounding
    b = f[0].copy()
    for i in range(1, 19):
        b = b + f[i]
    x = f.astype(np.longdouble)
    j = [sum(C[i][a] * x[i] for i in range(19)) for a in range(3)]
    m = [[j[a] * j[k] / b for k in range(3)] for a in range(3)]
    tr = m[0][0] + m[1][1] + m[2][2]
    errs = []
    for i in range(1, 19, 2):
        c = C[i]
        cmc = sum(c[a] * c[k] * m[a][k] for a in range(3) for k in range(3))
        q = (b + np.longdouble(4.5) * (cmc - tr / 3)).astype(np.float64)
        pair = star[i].astype(np.longdouble) + star[i + 1]
        errs.append((pair - 2 * np.longdouble(W[i]) * q) / np.spacing(W[i] * q))
    assert np.sqrt(np.mean(np.square(np.stack(errs)))) < 0.55
