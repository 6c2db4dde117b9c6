"""Units of length far from 1: the near/far test of tile boxes works in FP32 squares, so a system whose
element diameter squared leaves FP32's range must still get the contact law on every touching pair.

Lengths are scaled by a power of two, which scales every FP64 operation of the pair law exactly:
forces and potential energy against the FP64 oracle at the same scale, at the bars of systems of
ordinary scale (1e-12, 1e-11 for forces under eqs. 4-6).
"""

import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_common import force_error, print_case, require_gpu

pytestmark = pytest.mark.gpu

SCALES = [2.0 ** -90, 2.0 ** -52, 2.0 ** 60, 2.0 ** 80]


def _scaled(n, scale):
    ic = synth.with_velocity_noise(synth.make_binary(n, 0.5, seed=n), 0.05, 3)
    p, v = ic.f32_as_f64()
    return dataclasses.replace(ic, pos=p * scale, vel=v, D1=ic.D1 * scale, D2=ic.D2 * scale), ic


def _law(ic, law, scale):
    if law == "contact":
        return {}
    kw = synth.paper_law_params(ic)
    # eps is a length; gamma V against G m^2 / r^2 takes a length to the minus fifth power
    return dict(kw, eps=kw["eps"] * scale, gamma=kw["gamma"] * scale ** -5)


@pytest.mark.parametrize("law", ["contact", "paper"])
@pytest.mark.parametrize("scale", SCALES)
def test_fp64_forces_at_any_scale(scale, law):
    nb = require_gpu()
    n = 3000
    ic, base = _scaled(n, scale)
    kw = _law(base, law, scale)
    print_case("forces at scale", scale, law)
    nb.nb_tile_override(n, n, nb.NB_FP64, 1, 1, law=nb.LAWS[law])  # one chunk: the symmetric kernel
    try:
        s = nb.System(ic.pos, ic.vel, ic.n1, G=ic.G, m=ic.m, dt=1e-4, D1=ic.D1, D2=ic.D2, q=ic.q,
                      mode="fp64", law=law, **{k: x for k, x in kw.items() if k != "law"})
    finally:
        nb.nb_tile_override(n, n, nb.NB_FP64, 0, 1, law=nb.LAWS[law])
    a = s.accelerations()
    s.close()
    if kw:
        ref = oracle.accel_paper(ic.pos, ic.vel, ic.n1, ic.G, ic.m, ic.D1, ic.D2, kw["eps"],
                                 kw["gamma"], kw["beta"])
    else:
        ref = oracle.accel(ic.pos, ic.n1, ic.G, ic.m, ic.D1, ic.D2)
    assert force_error(a, ref) <= (1e-11 if kw else 1e-12)


@pytest.mark.parametrize("law", ["contact", "paper"])
@pytest.mark.parametrize("mode", ["kahan", "fp64"])
@pytest.mark.parametrize("scale", SCALES)
def test_potential_energy_at_any_scale(scale, mode, law):
    nb = require_gpu()
    if mode == "kahan" and law == "paper" and scale < 1.0:
        pytest.skip("refused: the overlap scale overflows FP32")
    ic, base = _scaled(3000, scale)
    kw = _law(base, law, scale)
    print_case("potential energy at scale", scale, mode, law)
    s = nb.System(ic.pos, ic.vel, ic.n1, G=ic.G, m=ic.m, dt=1e-4, D1=ic.D1, D2=ic.D2, q=ic.q,
                  mode=mode, law=law, **{k: x for k, x in kw.items() if k != "law"})
    pe = s.diagnostics(with_pe=True)["PE"]
    s.close()
    if kw:
        ref = oracle.paper_pe(ic.pos, ic.n1, ic.G, ic.m, ic.D1, ic.D2, kw["eps"], kw["gamma"])
    else:
        ref = oracle.diag(ic.pos, np.zeros_like(ic.pos), ic.n1, ic.G, ic.m, ic.D1, ic.D2)["PE"]
    assert abs(pe - ref) <= 1e-12 * abs(ref)
