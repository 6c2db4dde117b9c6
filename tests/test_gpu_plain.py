"""The plain FP32 force kernel: one running sum per element over all j in sorted order, the real
elements packed into waves (one wave may hold the end of one star and the start of the other).

Sizes with a star boundary inside a wave, at its edge and at a tile's edge, stars of one element,
few and many workgroups (the kernel's two forms), against the oracle at the mode's 1e-4 of small
systems (3e-5 is its error at 131,072 elements), and bitwise the same alone and in a batch."""

import numpy as np
import pytest

import oracle
import synth
from gpu_common import force_error, print_case, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n1", [(1, 1), (2, 1), (65, 64), (300, 255), (600, 256), (1000, 321),
                                  (1024, 512), (4097, 4096), (5003, 1), (70000, 41999)])
def test_plain_forces_and_batch(n, n1):
    nb = require_gpu()
    ic = synth.make_binary(n, 1.0, seed=n)
    p, v = ic.f32()
    D1, D2 = ic.D1, 0.8 * ic.D1
    kw = dict(G=1.0, m=ic.m, dt=1e-4, D1=D1, D2=D2, q=0.7, mode="plain")
    print_case("plain forces", n, n1)
    s, t = nb.System(p, v, n1, **kw), nb.System(p, v, n1, **kw)
    u = nb.System.from_ic(synth.make_binary(777, 0.4, seed=1), mode="plain")
    a = s.accelerations()
    rows = np.unique(np.r_[0:min(n, 400), max(0, n1 - 70):min(n, n1 + 70), max(0, n - 300):n])
    ref = oracle.accel(p.astype(np.float64), n1, 1.0, ic.m, D1, D2, rows=rows)
    assert force_error(a[rows], ref) <= 1e-4
    s.step(3)
    nb.step_many([u, t], 3)
    assert np.array_equal(s.positions(), t.positions())
    assert np.array_equal(s.accelerations(), t.accelerations())
    for x in (s, t, u):
        x.close()
