"""The Courant step and the div B monitor have kernels of their own: the speeds
are those the face-flux pass reports, and the div B pass, which walks up to eight
planes a thread on large grids, agrees with the oracle at its seams."""

import numpy as np
import pytest

from problems import fields
import oracle
import problems

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make", [
    lambda r, p: problems.fm_torus(n1=61, n2=29, n3=5, recon=r, precision=p),
    lambda r, p: problems.fm_torus(n1=186, n2=63, n3=45, recon=r, precision=p),  # large blocks
    lambda r, p: (lambda prm, P0: (dict(prm, recon=r, precision=p), P0))(*problems.cks_bondi(33, 20, 11)),
], ids=["torus_61x29x5", "torus_186x63x45", "cks_33x20x11"])
@pytest.mark.parametrize("recon,precision", [
    (problems.RECON_MC, problems.FP64), (problems.RECON_WENO5, problems.FP64),
    (problems.RECON_MC, problems.MIXED), (problems.RECON_WENO5, problems.MIXED)],
    ids=["mc_fp64", "weno5_fp64", "mc_mixed", "weno5_mixed"])
def test_speeds_alone_are_those_of_the_fluxes(lib, make, recon, precision):
    """Bit for bit, and a state whose signal speed is not finite (the coarse torus
    with MC slopes in single-precision fluxes has one) is refused after either."""
    def speeds():
        try:
            return lib.grmhd_speeds(sim.ctx)
        except lib.GrmhdError as e:
            return str(e)

    prm, P0 = make(recon, precision)
    sim = lib.Sim(prm)
    P = sim.to_device(P0)
    try:
        dt = sim.get_dt(P)
    except lib.GrmhdError:
        dt = None
    alone = speeds()
    lib.grmhd_substep(sim.ctx, P, P, P.clone(), 0.01, want_speeds=True)
    assert speeds() == alone
    assert (dt is None) == isinstance(alone, str)
    if dt is not None:
        assert all(np.isfinite(alone)) and dt == lib.grmhd_courant_dt(sim.ctx, [alone])
    sim.close()


MODES = ((1, 1, 1.0, 3), (2, 1, 0.7, 1), (2, 2, 0.35, 0), (3, 1, 0.4, 2))


@pytest.mark.parametrize("make", [
    lambda: fields.sine_box(5, 3, 1, ((1, 1, 1.0, 0), (2, 1, 0.5, 0))),
    lambda: fields.sine_box(64, 64, 131, MODES),   # two planes a thread, one over
    lambda: fields.sine_box(130, 132, 85, MODES),  # eight planes a thread, five over
    lambda: fields.sine_kerr(n1=130, n2=132, n3=85, m=2, c=0.3),
], ids=["box_5x3x1", "box_64x64x131", "box_130x132x85", "kerr_130x132x85"])
def test_divb_matches_oracle_where_threads_walk(lib, make):
    """to 1e-12 relative, as for the small grids: two dozen terms of the result's
    size, rounded to 1e-16 each, in another association than the oracle's"""
    prm, P0, div = make()
    want = float(np.abs(div).max())
    ref = oracle.divb(P0, oracle.Grid(prm))
    sim = lib.Sim(prm)
    P = sim.to_device(P0)
    got = [sim.divb(P), sim.divb(0.5 * P), lib.grmhd_divb_noalloc(sim.ctx, P)]
    sim.close()
    assert got[0] == got[2] and got[1] == 0.5 * got[0]
    assert abs(got[0] / ref - 1.0) < 1e-12 and abs(got[0] / want - 1.0) < 1e-12, (got, ref, want)
