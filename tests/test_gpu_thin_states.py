"""Signal speeds of thin states in mixed precision: the faces' speeds are
quotients of densities, so they neither lose nor gain by the densities' scale.
The magnetosonic speed's square is q / (m + q) times a metric factor; a product
of the two densities would leave the normal range of FP32 near 1e-19."""

import numpy as np
import pytest

import problems

pytestmark = pytest.mark.gpu
NG = 3
# some 20 FP32 operations of 2^-24 = 6e-8 a speed, half of them under the root
TOL = 2e-6


def speeds(lib, prm, P0, precision):
    sim = lib.Sim(dict(prm, precision=precision))
    P = sim.to_device(P0)
    dt = sim.get_dt(P)
    out = np.array([*lib.grmhd_speeds(sim.ctx), dt])
    sim.close()
    return out


def scaled_box(recon, scale):
    prm, P0 = problems.linear_modes(n=24, recon=recon)
    P0 = P0.copy()
    P0[:2] *= scale
    P0[5:] *= scale ** 0.5
    return prm, P0


def atmosphere(recon, scale):
    """rho and u at their floors, at rest, at 800 < r < 1000 about the midplane
    (rho 1e-14 to 2e-14, u 3e-20 to 7e-20 at scale 1)"""
    torus, _ = problems.fm_torus(n1=16, n2=8, n3=1)
    dirichlet = [problems.BC_DIRICHLET] * 2
    prm = dict(torus, n1=32, n2=16, n3=8, recon=recon, x1min=np.log(800.0), x1max=np.log(1000.0), x2min=0.45, x2max=0.55,
               bc=[dirichlet, dirichlet, torus["bc"][2]])
    r = np.exp(prm["x1min"] + (np.arange(-NG, prm["n1"] + NG) + 0.5) * (prm["x1max"] - prm["x1min"]) / prm["n1"])
    k = scale / (r * r * (1.0 + r / 10.0))
    P0 = np.zeros((8, prm["n3"] + 2 * NG, prm["n2"] + 2 * NG, prm["n1"] + 2 * NG))
    P0[0] = prm["rho_fl"] * k
    P0[1] = prm["u_fl"] * (k / scale) ** prm["gam"] * scale
    return prm, P0


@pytest.mark.parametrize("make,scale,recon", [
    (make, scale, recon) for recon in (problems.RECON_MC, problems.RECON_WENO5)
    for make, scale in ((scaled_box, 1e-16), (scaled_box, 1e-20), (scaled_box, 1e-24), (atmosphere, 1.0), (atmosphere, 1e-6))
    # at 1e-26, differences of u are below what the FP32 limiter's product of two holds
    if (make, scale, recon) != (atmosphere, 1e-6, problems.RECON_MC)],
    ids=lambda v: {problems.RECON_MC: "mc", problems.RECON_WENO5: "weno5"}[v] if isinstance(v, int) else
    v if isinstance(v, float) else v.__name__)
def test_mixed_speeds_of_thin_states_are_those_of_fp64(lib, make, scale, recon):
    prm, P0 = make(recon, scale)
    want = speeds(lib, prm, P0, problems.FP64)
    got = speeds(lib, prm, P0, problems.MIXED)
    assert (want > 0.0).all(), want
    assert (np.abs(got / want - 1.0) < TOL).all(), (got, want)
