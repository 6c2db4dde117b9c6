"""System() from host arrays that may not be written to (a memory map, a broadcast, a frozen array): taken
as they are, without a warning, with the state of a plain copy."""

import warnings

import numpy as np
import pytest

import synth
from gpu_common import print_case, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["kahan", "fp64"])
def test_read_only_arrays(mode, tmp_path):
    nb = require_gpu()
    print_case("read-only inputs", mode)
    ic = synth.make_binary(700, 0.5, seed=1)
    p, v = ic.f32() if mode == "kahan" else ic.f32_as_f64()
    kw = dict(G=ic.G, m=ic.m, dt=1e-4, D1=ic.D1, D2=ic.D2, q=ic.q, mode=mode)
    np.save(tmp_path / "p.npy", p)
    frozen = v.copy()
    frozen.setflags(write=False)
    want = nb.System(p.copy(), v.copy(), ic.n1, **kw)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        got = nb.System(np.load(tmp_path / "p.npy", mmap_mode="r"), frozen, ic.n1, **kw)
        still = nb.System(p.copy(), np.broadcast_to(np.zeros(3, p.dtype), p.shape), ic.n1, **kw)
    for f in ("positions", "velocities", "accelerations"):
        assert np.array_equal(getattr(got, f)(), getattr(want, f)())
    assert not still.velocities().any()
    for s in (want, got, still):
        s.close()
