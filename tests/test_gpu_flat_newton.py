"""A Newton derivative of exactly zero in the 1D_W inversion: the step is -inf, so
W is halved, and the iteration goes on to the root below (as the oracle's, which
divides in IEEE arithmetic). The case: at W = 1, v^2 = 3/4 and D = 5/16 every
operation of the derivative is exact, and with 1/gamma_frac = 41/32 it is 1 - 1;
the energy is that of the root at W = 0.95."""

import numpy as np
import pytest

import oracle
import problems

pytestmark = pytest.mark.gpu
NG = 3


def test_inversion_from_a_guess_with_zero_derivative(lib):
    D, gam = 0.3125, 1.28125 / (1.28125 - 1.0)
    gf = (gam - 1.0) / gam
    assert gf * 1.28125 == 1.0
    prm = problems.base_problem(4, 4, 4, gam=gam)
    W = 0.95
    v2 = 0.75 / W ** 2
    s = np.sqrt(1.0 - v2)
    U = np.zeros((8, 4, 4, 4))
    U[0] = D
    U[1] = -((W - D) - gf * ((W - D) * (1.0 - v2) - D * s * v2 / (1.0 + s)))
    U[2:5] = 0.5
    guess = np.zeros((8, 4, 4, 4))
    guess[0] = 1.0                  # W = rho at rest
    ref, failed = oracle.cons_to_prim(U, guess, oracle.Grid(prm))
    assert not failed.any() and ref[1].min() > 0.0
    sim = lib.Sim(prm)
    pad = ((0, 0), (NG, NG), (NG, NG), (NG, NG))
    Ud, Pd = sim.to_device(np.pad(U, pad)), sim.to_device(np.pad(guess, pad))
    assert sim.cons_to_prim(Ud, Pd) == 0
    got = sim.to_host(Pd)[:, NG:-NG, NG:-NG, NG:-NG]
    sim.close()
    assert np.abs(got / np.where(ref == 0.0, 1.0, ref) - (ref != 0.0)).max() < 1e-12
