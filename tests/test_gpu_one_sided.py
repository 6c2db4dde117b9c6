"""The one-sided force kernel of small systems (the finest split of at most a few thousand elements,
FP32 Kahan and FP64 modes) and the pass between two evaluations.

Sizes at the edges of a workgroup's elements (8 in FP32, 4 in FP64), of the 256 lanes that share
the j and of the largest such system, one star empty or of one element, both element laws:
forces against the oracle at the bars of the other kernels (1e-5 FP32; 1e-12 FP64, 1e-11 under
eqs. 4-6), against the symmetric kernel of the same system (a coarser split), and in a batch with
systems of the other kernels bitwise as alone.
"""

import numpy as np
import pytest

import oracle
import synth
from gpu_common import force_error, print_case, require_gpu

pytestmark = pytest.mark.gpu

BAR = {("kahan", "contact"): 1e-5, ("kahan", "paper"): 1e-5, ("fp64", "contact"): 1e-12,
       ("fp64", "paper"): 1e-11}


def _system(nb, ic, mode, law):
    kw = synth.paper_law_params(ic) if law == "paper" else {}
    return nb.System.from_ic(ic, mode=mode, **kw), kw


def _oracle(ic, kw, D2=None):
    p, v = ic.f32_as_f64()
    D2 = ic.D2 if D2 is None else D2
    if kw:
        return oracle.accel_paper(p, v, ic.n1, ic.G, ic.m, ic.D1, D2, kw["eps"], kw["gamma"],
                                  kw["beta"])
    return oracle.accel(p, ic.n1, ic.G, ic.m, ic.D1, D2)


@pytest.mark.parametrize("mode,law", list(BAR))
@pytest.mark.parametrize("n,q", [(1, 0.5), (2, 1.0), (9, 0.5), (17, 0.07), (255, 0.3),
                                 (258, 0.004), (1023, 1.0), (1025, 0.6), (3077, 0.8),
                                 (8192, 0.3)])
def test_forces_match_oracle(n, q, mode, law):
    nb = require_gpu()
    ic = synth.with_velocity_noise(synth.make_binary(n, q, seed=n), 0.05, 3)
    print_case("one-sided forces", n, q, mode, law)
    M, W = nb.MODES[mode], nb.LAWS[law]
    nb.nb_tile_override(n, n, M, 4096, 1, law=W)  # one tile per chunk
    try:
        s, kw = _system(nb, ic, mode, law)
        need = nb.nb_scratch_bytes(s.params)
        nb.nb_tile_override(n, n, M, 1, 1, law=W)  # one chunk: the symmetric kernel from two tiles on
        t, _ = _system(nb, ic, mode, law)
        coarse = nb.nb_scratch_bytes(t.params)
    finally:
        nb.nb_tile_override(n, n, M, 0, 1, law=W)
    if n > 256:
        assert need != coarse  # two kernels, two layouts
    a, b = s.accelerations(), t.accelerations()
    s.forces()
    assert np.array_equal(s.accelerations(), a)
    s.close()
    t.close()
    ref = _oracle(ic, kw)
    assert force_error(a, ref) <= BAR[mode, law]
    assert force_error(a, b.astype(np.float64)) <= 2 * BAR[mode, law]


@pytest.mark.parametrize("mode,law", list(BAR))
def test_batch_with_other_kernels_equals_alone(mode, law):
    """One-sided systems with larger ones (bands, a system of many units) and an empty one in one
    table: bitwise as alone, through nb_step, a graph and nb_step_static, over calls of one and
    of several steps; the run follows the oracle's counts."""
    nb = require_gpu()
    sizes = [(700, 0.9), (9000, 0.5), (2048, 0.5), (30000, 0.3), (5003, 0.2), (66000, 0.4)]
    if mode == "fp64":
        sizes = sizes[:4]
    print_case("one-sided in a batch", mode, law)

    def make():
        return [_system(nb, synth.with_velocity_noise(synth.make_binary(n, q, seed=n, R2=0.45),
                                                      2.0, 5), mode, law)[0] for n, q in sizes]

    alone, mix, graph, sta = make(), make(), make(), make()
    empty = nb.System(np.zeros((0, 3)), np.zeros((0, 3)), 0, G=1.0, m=1.0, dt=1e-4, D1=0.1, D2=0.1,
                      q=0.5, mode=mode, **({"law": "paper", "gamma": 1.0} if law == "paper" else {}))
    for s in alone:
        s.step(1)
        s.step(5)
    nb.step_many([empty] + mix, 1)
    nb.step_many(mix + [empty], 5)
    g = nb.nb_graph_create([s.handle for s in graph], 3, graph[0].stream)
    for _ in range(2):
        nb.nb_graph_launch(g, graph[0].stream)
        graph[0].synchronize()
    nb.nb_graph_destroy(g)
    nb.nb_step_static([s.handle for s in sta], 6, sta[0].stream)
    assert empty.diagnostics()["step"] == 6
    crossings = 0
    for k, (n, q) in enumerate(sizes):
        log = alone[k].l1_log()
        crossings += int(log[:, 2:].sum())
        assert log[:, 0].tolist() == list(range(1, 7))
        for other in (mix, graph, sta):
            for f in ("positions", "velocities", "accelerations", "sides", "l1_log"):
                assert np.array_equal(getattr(other[k], f)(), getattr(alone[k], f)()), (n, f)
            d, e = other[k].diagnostics(), alone[k].diagnostics()
            assert all(np.array_equal(d[key], e[key]) for key in d), n
    assert crossings > 0
    for s in alone + mix + graph + sta + [empty]:
        s.close()


@pytest.mark.parametrize("mode,law", list(BAR))
@pytest.mark.parametrize("n,q", [(700, 0.4), (2048, 0.5), (2801, 0.9), (3501, 0.2), (3802, 0.6),
                                 (4501, 0.7), (6401, 0.3)])
def test_elements_per_workgroup(n, q, mode, law):
    """Sizes at which a workgroup takes 4 to 8 elements (FP64: 2 to 4), with remainders in both stars:
    the forces, and those that a step leaves, against the oracle at the step's own positions."""
    nb = require_gpu()
    ic = synth.with_velocity_noise(synth.make_binary(n, q, seed=n), 0.05, 3)
    print_case("elements per workgroup", n, q, mode, law)
    M, W = nb.MODES[mode], nb.LAWS[law]
    nb.nb_tile_override(n, n, M, 4096, 1, law=W)
    try:
        s, kw = _system(nb, ic, mode, law)
    finally:
        nb.nb_tile_override(n, n, M, 0, 1, law=W)
    a = s.accelerations()
    ref = _oracle(ic, kw)
    assert force_error(a, ref) <= BAR[mode, law]
    s.step(1)
    after = s.accelerations()
    p = np.stack([c.cpu().numpy().astype(np.float64) for c in (s.x, s.y, s.z)], axis=1)
    assert not np.array_equal(p, ic.f32_as_f64()[0])
    s.close()
    if kw:  # the force of the step takes the half-step velocities, which no array holds
        return
    assert force_error(after, oracle.accel(p, ic.n1, ic.G, ic.m, ic.D1, ic.D2)) <= BAR[mode, law]


BARS = {"kahan": (1e-5, 1e-4), "fp64": (1e-11, 1e-10)}  # positions (of a), velocities (of max|v|)
LIMIT = {("kahan", "contact"): 7168, ("kahan", "paper"): 7168, ("fp64", "contact"): 4096,
         ("fp64", "paper"): 2560}


@pytest.mark.parametrize("mode,law", list(BAR))
@pytest.mark.parametrize("past", [0, 1])
def test_runs_at_the_limit_follow_the_oracle(mode, law, past):
    """The largest one-sided system and the smallest beyond it, in the finest split: forces, a run of
    twelve steps against the oracle's, and the L1 counts of every step against the oracle's count of
    the same positions; stepping one by one and in one call gives the same bits."""
    nb = require_gpu()
    n = LIMIT[mode, law] + past
    ic = synth.with_velocity_noise(synth.make_binary(n, 0.5, seed=n, R2=0.45), 2.0, 5)
    print_case("at the limit", n, mode, law)
    M, W = nb.MODES[mode], nb.LAWS[law]
    nb.nb_tile_override(n, n, M, 4096, 1, law=W)
    try:
        s, kw = _system(nb, ic, mode, law)
        t, _ = _system(nb, ic, mode, law)
    finally:
        nb.nb_tile_override(n, n, M, 0, 1, law=W)
    assert force_error(s.accelerations(), _oracle(ic, kw)) <= BAR[mode, law]
    side = np.zeros(n, dtype=np.int8)
    oracle.l1_count(s.positions().astype(np.float64), ic.n1, ic.q, side, init=True)
    want = []
    for k in range(12):
        s.step(1)
        want.append((k + 1, *oracle.l1_count(s.positions().astype(np.float64), ic.n1, ic.q, side)))
    t.step(12)
    assert s.l1_log().tolist() == t.l1_log().tolist() == [list(w) for w in want]
    for f in ("positions", "velocities", "accelerations", "sides"):
        assert np.array_equal(getattr(s, f)(), getattr(t, f)()), f
    p, v = ic.f32_as_f64()
    law_kw = dict(law=1, eps=kw["eps"], gamma=kw["gamma"], beta=kw["beta"]) if kw else {}
    run = oracle.Run(p, v, ic.n1, ic.G, ic.m, 1e-4, ic.D1, ic.D2, ic.q, a=ic.a, R2_0=ic.R2, **law_kw)
    run.advance(12)
    xtol, vtol = BARS[mode]
    if mode == "kahan" and kw:
        vtol = 2e-3  # a pair near a sign tie may take the other branch for a step
    assert t.diagnostics()["D2"] == run.D2
    assert np.abs(t.positions() - run.pos).max() <= xtol * ic.a
    assert np.abs(t.velocities() - run.vel).max() <= vtol * np.abs(run.vel).max()
    s.close()
    t.close()


@pytest.mark.parametrize("mode,law", list(BAR))
def test_batch_of_one_sided_systems_follows_the_oracle(mode, law):
    """One-sided systems with larger ones in one table, twelve steps in one call: every system's run and
    D2 against its own oracle run, and its L1 record of every step exactly in FP64."""
    nb = require_gpu()
    sizes = [(700, 0.9), (9000, 0.5), (2048, 0.5), (1203, 0.2)]
    print_case("one-sided batch against the oracle", mode, law)
    ics = [synth.with_velocity_noise(synth.make_binary(n, q, seed=n, R2=0.45), 2.0, 5)
           for n, q in sizes]
    made = [_system(nb, ic, mode, law) for ic in ics]
    nb.step_many([s for s, _ in made], 12)
    xtol, vtol = BARS[mode]
    for (s, kw), ic in zip(made, ics):
        p, v = ic.f32_as_f64()
        law_kw = dict(law=1, eps=kw["eps"], gamma=kw["gamma"], beta=kw["beta"]) if kw else {}
        run = oracle.Run(p, v, ic.n1, ic.G, ic.m, 1e-4, ic.D1, ic.D2, ic.q, a=ic.a, R2_0=ic.R2,
                         **law_kw)
        counts, _ = run.advance(12)
        assert s.diagnostics()["D2"] == run.D2
        assert np.abs(s.positions() - run.pos).max() <= xtol * ic.a
        tol = 2e-3 if mode == "kahan" and kw else vtol
        assert np.abs(s.velocities() - run.vel).max() <= tol * np.abs(run.vel).max()
        if mode == "fp64":
            assert np.array_equal(s.l1_log()[:, 1:], counts)
        s.close()


@pytest.mark.parametrize("mode", ["kahan", "fp64"])
@pytest.mark.parametrize("n,q", [(700, 0.4), (1203, 0.9), (2048, 0.5), (2551, 0.6), (3501, 0.2),
                                 (6401, 0.3)])
def test_elements_per_workgroup_in_a_step_of_the_paper_law(n, q, mode):
    """The forces that a step under eqs. (4)-(6) leaves, at the sizes of the different elements per
    workgroup. They take the step's half-step velocities, v - a dt/2 of the state it leaves: in FP64
    rounded once more, which the bar of 1e-11 holds; in FP32 a run of one step against the oracle's
    at the bars of a trajectory."""
    nb = require_gpu()
    if mode == "fp64" and n > LIMIT["fp64", "paper"]:
        pytest.skip("not one-sided")
    ic = synth.with_velocity_noise(synth.make_binary(n, q, seed=n), 0.05, 3)
    print_case("elements per workgroup, step of eqs. (4)-(6)", n, q, mode)
    M, W = nb.MODES[mode], nb.LAWS["paper"]
    nb.nb_tile_override(n, n, M, 4096, 1, law=W)
    try:
        s, kw = _system(nb, ic, mode, "paper")
    finally:
        nb.nb_tile_override(n, n, M, 0, 1, law=W)
    s.step(1)
    p, v, a = (x.astype(np.float64) for x in (s.positions(), s.velocities(), s.accelerations()))
    D2 = s.diagnostics()["D2"]
    s.close()
    p0, v0 = ic.f32_as_f64()
    run = oracle.Run(p0, v0, ic.n1, ic.G, ic.m, 1e-4, ic.D1, ic.D2, ic.q, a=ic.a, R2_0=ic.R2, law=1,
                     eps=kw["eps"], gamma=kw["gamma"], beta=kw["beta"])
    run.advance(1)
    assert D2 == run.D2
    assert np.abs(p - run.pos).max() <= BARS[mode][0] * ic.a
    assert np.abs(v - run.vel).max() <= (2e-3 if mode == "kahan" else 1e-10) * np.abs(run.vel).max()
    if mode == "fp64":
        half = v - a * 0.5e-4
        ref = oracle.accel_paper(p, half, ic.n1, ic.G, ic.m, ic.D1, ic.D2, kw["eps"], kw["gamma"],
                                 kw["beta"])
        assert force_error(a, ref) <= BAR[mode, "paper"]
