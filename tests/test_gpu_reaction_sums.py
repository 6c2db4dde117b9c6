"""How the symmetric kernel sums the reactions of a band of rows in FP32.

All elements of star 1 at one point and star 2's on a cap about it: every term of a reaction on an
element of star 2 is the same number t, and a running FP32 sum of m equal terms, m t, is off by
up to sum_{k=2..m} u k t = (m + 1) u / 2 of it (u = 2^-24) and, for some t, by half of that. The
kernel adds runs of at most 128 terms, so its forces stay within 64.5 u of the largest force, plus
16 u for a term's own rounding (u in the square, 2 u in the reciprocal root, thrice that and 2 u in
its cube, u in the product) and for the few sums of runs and bands. One run over a band of two
rows (512 terms) misses this bar by half.
"""

import numpy as np
import pytest

import oracle
from gpu_common import force_error, print_case, require_gpu

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.mark.parametrize("rows", [2, 4])
def test_long_reaction_sums(rows):
    nb = require_gpu()
    n1, n2 = 4096, 64
    n = n1 + n2
    rng = np.random.default_rng(7)
    # on a grid: a close pair among them would set the scale of the forces
    y, z = np.meshgrid(np.linspace(-0.2, 0.2, 8), np.linspace(-0.2, 0.2, 8))
    cap = np.column_stack([1.0 + rng.uniform(0.0, 1e-3, n2), y.ravel(), z.ravel()])
    pos = np.concatenate([np.zeros((n1, 3)), cap]).astype(np.float32)
    print_case("reaction sums", rows)
    kw = dict(G=1.0, m=1.0 / n1, dt=1e-4, D1=1e-3, D2=1e-3, q=0.5)
    nb.nb_tile_override(n, n, nb.NB_FP32_KAHAN, 1, rows)
    try:
        s = nb.System(pos, np.zeros_like(pos), n1, mode="kahan", **kw)
    finally:
        nb.nb_tile_override(n, n, nb.NB_FP32_KAHAN, 0, 1)
    a = s.accelerations()
    s.close()
    ref = oracle.accel(pos.astype(np.float64), n1, kw["G"], kw["m"], kw["D1"], kw["D2"])
    err = force_error(a, ref)
    print("rows", rows, "error", err)
    assert err <= (64.5 + 16) * U
