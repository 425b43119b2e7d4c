"""Rounding: the inversion is no further from the oracle in 80-bit arithmetic than
the oracle in 64 bits is, corrected reciprocals and roots in place of IEEE
divisions notwithstanding."""

import numpy as np
import pytest

import oracle
import problems

LD = np.longdouble
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(np.finfo(LD).nmant < 63, reason="needs an 80-bit long double")]
NG = 3
# 110592 rounding errors a side (24^3 zones, 8 variables): the two norms' ratio
# scatters by well under a percent where the errors are alike
BAR = 1.05


def interior(P, prm):
    return P[:, NG:NG + prm["n3"], NG:NG + prm["n2"], NG:NG + prm["n1"]]


def norms(got, own, true):
    err = lambda a: float(np.sqrt(((a - true) ** 2).sum() / (true ** 2).sum()))
    assert true.dtype == LD
    return err(got.astype(LD)), err(own.astype(LD))


def test_inversion_rounds_as_ieee_arithmetic_does(lib):
    prm, P0 = problems.linear_modes(n=24, amp=1e-2)
    g = oracle.Grid(prm)
    U = oracle.prim_to_cons(P0, g)
    guess = interior(P0, prm) * np.array([1.01, 0.97, 0.9, 0.9, 0.9, 1, 1, 1]).reshape(8, 1, 1, 1)
    own, _ = oracle.cons_to_prim(U, guess, g)
    true, _ = oracle.cons_to_prim(U.astype(LD), guess.astype(LD), g)
    sim = lib.Sim(prm)
    pad = ((0, 0), (NG, NG), (NG, NG), (NG, NG))
    Ud, Pd = sim.to_device(np.pad(U, pad)), sim.to_device(np.pad(guess, pad))
    assert sim.cons_to_prim(Ud, Pd) == 0
    here, ieee = norms(interior(sim.to_host(Pd), prm), own, true)
    sim.close()
    print("inversion: GPU %.3e, oracle %.3e" % (here, ieee))
    assert here <= BAR * ieee
