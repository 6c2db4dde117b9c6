"""nb_set_force_grid with small (one-sided) systems: the bound on the launch's workgroups holds for them,
and steps of a batch that mixes them with systems in bands of one, two and four rows and an empty
one are bitwise those of the default launch, alone and together, over calls of one and several steps.
"""

import numpy as np
import pytest

import synth
from gpu_common import print_case, require_gpu

pytestmark = pytest.mark.gpu

CASES = [("kahan", "contact"), ("kahan", "paper"), ("fp64", "contact"), ("fp64", "paper")]


def _make(nb, n, q, mode, law):
    ic = synth.with_velocity_noise(synth.make_binary(n, q, seed=n, R2=0.45), 2.0, 5)
    return nb.System.from_ic(ic, mode=mode, **(synth.paper_law_params(ic) if law == "paper" else {}))


@pytest.mark.parametrize("mode,law", CASES)
@pytest.mark.parametrize("blocks", [3, 64, 100000])
def test_steps_under_a_persistent_launch(blocks, mode, law):
    nb = require_gpu()
    print_case("force grid", blocks, mode, law)
    sizes = [(700, 0.9), (2048, 0.5), (9000, 0.5), (1, 0.5), (12001, 0.3), (1203, 0.2)]
    rows = {9000: 2, 12001: 4} if mode == "kahan" else {}
    M, W = nb.MODES[mode], nb.LAWS[law]
    empty_kw = {"law": "paper", "gamma": 1.0} if law == "paper" else {}

    def run():
        for n, r in rows.items():
            nb.nb_tile_override(n, n, M, 8, r, law=W)
        try:
            S = [_make(nb, n, q, mode, law) for n, q in sizes]
        finally:
            for n in rows:
                nb.nb_tile_override(n, n, M, 0, 1, law=W)
        z = np.zeros((0, 3))
        S.append(nb.System(z, z, 0, G=1.0, m=1.0, dt=1e-4, D1=0.1, D2=0.1, q=0.5, mode=mode, **empty_kw))
        S[0].step(1)
        S[1].step(3)
        nb.step_many(S, 1)
        nb.step_many(S, 4)
        S[2].forces()
        S[1].forces()
        out = [[getattr(s, f)() for f in ("positions", "velocities", "accelerations", "sides", "l1_log")]
               for s in S]
        d = [s.diagnostics() for s in S]
        for s in S:
            s.close()
        return out, d

    want, wd = run()
    nb.nb_set_force_grid(blocks)
    try:
        got, gd = run()
    finally:
        nb.nb_set_force_grid(0)
    for a, b in zip(want, got):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    for a, b in zip(wd, gd):
        assert all(np.array_equal(a[k], b[k]) for k in a)


@pytest.mark.parametrize("step", [False, True])
def test_one_workgroup_runs_one_compute_units_worth(step):
    """Bounded to one workgroup, the some 900 of 7,001 elements run one after the other on one of the
    chip's 256 compute units: at least eight times the default launch's time, whatever overlaps."""
    nb = require_gpu()
    print_case("force grid of one", step)
    s = _make(nb, 7001, 0.5, "kahan", "contact")

    def ms(blocks):
        nb.nb_set_force_grid(blocks)
        try:
            s.forces()
            s.synchronize()
            nb.nb_timing_reset()
            nb.nb_timing_enable(True)
            s.step(2) if step else s.forces()
            nb.nb_timing_enable(False)
            return nb.nb_timing_read()[0]
        finally:
            nb.nb_timing_enable(False)
            nb.nb_set_force_grid(0)

    default, bounded = ms(0), ms(1)
    nb.nb_timing_reset()
    s.close()
    print("default %.4f ms, one workgroup %.4f ms" % (default, bounded))
    assert bounded >= 8 * default
