"""The potential energy of nb_diagnostics: every unordered pair once, over tiles of 256 sorted
slots, with a form of its own for tiles whose boxes are at least D apart.

Sizes at the edges of tiles and of the split, dense and compact stars (most tiles near), both
element laws and the FP32 and FP64 states, against the FP64 oracle on the same positions at the
1e-12 that sums of FP64 pair terms are held to; elements that coincide, or whose position is not
finite, add nothing.
"""

import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_common import print_case, require_gpu

pytestmark = pytest.mark.gpu

TOL = 1e-12


def _oracle_pe(ic, pos, n1, kw):
    if kw:
        return oracle.paper_pe(pos, n1, ic.G, ic.m, ic.D1, ic.D2, kw["eps"], kw["gamma"])
    return oracle.diag(pos, np.zeros_like(pos), n1, ic.G, ic.m, ic.D1, ic.D2)["PE"]


def _kw(ic, law):
    return synth.paper_law_params(ic) if law == "paper" else {}


@pytest.mark.parametrize("law", ["contact", "paper"])
@pytest.mark.parametrize("mode", ["kahan", "fp64", "plain"])
@pytest.mark.parametrize("n,q,R1", [(2, 1.0, 0.3), (255, 0.02, 0.3), (257, 0.5, 0.3),
                                    (513, 1.0, 0.05), (1001, 0.3, 0.3), (2600, 0.9, 0.02),
                                    (23300, 0.5, 0.3)])
def test_potential_energy_matches_oracle(n, q, R1, mode, law):
    nb = require_gpu()
    if mode == "plain" and law == "paper":
        pytest.skip("the plain mode has no such law")
    ic = synth.make_binary(n, q, seed=n, R1=R1)
    kw = _kw(ic, law)
    print_case("potential energy", n, q, R1, mode, law)
    s = nb.System.from_ic(ic, mode=mode, **kw)
    pe = s.diagnostics(with_pe=True)["PE"]
    again = s.diagnostics(with_pe=True)["PE"]
    s.close()
    ref = _oracle_pe(ic, ic.f32_as_f64()[0], ic.n1, kw)
    assert pe == again
    assert abs(pe - ref) <= TOL * abs(ref)


@pytest.mark.parametrize("law", ["contact", "paper"])
@pytest.mark.parametrize("mode", ["kahan", "fp64"])
def test_coincident_and_non_finite_elements_add_nothing(mode, law):
    nb = require_gpu()
    ic = synth.make_binary(700, 0.5, seed=3)
    pos = ic.f32_as_f64()[0]
    pos[11] = pos[10]  # star 1, and one across the stars
    pos[600] = pos[20]
    ic = dataclasses.replace(ic, pos=pos)
    kw = _kw(ic, law)
    print_case("potential energy, degenerate elements", mode, law)
    s = nb.System.from_ic(ic, mode=mode, **kw)
    ref = _oracle_pe(ic, pos, ic.n1, kw)
    assert abs(s.diagnostics(with_pe=True)["PE"] - ref) <= TOL * abs(ref)
    s.x[5], s.y[650], s.z[300] = float("nan"), float("inf"), float("-inf")
    pe = s.diagnostics(with_pe=True)["PE"]
    s.close()
    kept = np.delete(np.arange(700), [5, 300, 650])
    ref = _oracle_pe(ic, pos[kept], int((kept < ic.n1).sum()), kw)
    assert abs(pe - ref) <= TOL * abs(ref)
