"""Each block shape of the face-flux pass, asked for by a tile, gives the same bits
on grids that its tiles fit exactly (14 and 28 zones in x1 for the 16-wide ones,
30 and 60 for 32, 62 and 124 for 64; 7 and 14 rows less one) and on one zone
more, on grids narrower than a tile and on a single plane."""

import numpy as np
import pytest

import problems

pytestmark = pytest.mark.gpu

SHAPES = [(128, 4), (32, 8), (16, 8)]   # large, small, narrow
MODES = [(problems.RECON_WENO5, problems.FP64), (problems.RECON_MC, problems.FP64),
         (problems.RECON_WENO5, problems.MIXED), (problems.RECON_MC, problems.MIXED)]
MODE_IDS = ["weno5_fp64", "mc_fp64", "weno5_mixed", "mc_mixed"]


def same(lib, prm, P0, electrons):
    out = []
    for tile in [None] + SHAPES:
        sim = lib.Sim(prm)
        if tile:
            sim.set_tiles("sweep", *tile)
        P = sim.to_device(P0)
        dt0 = sim.get_dt(P)
        if electrons:
            E = sim.to_device(problems.electron_scalars(P0, prm["gam"]))
            dt = sim.run_electrons(P, E, 2, dt0, "constant", 0.5)
            out.append((dt0, dt, sim.to_host(P), sim.to_host(E)))
        else:
            out.append((dt0, sim.run(P, 2, dt0), sim.to_host(P), np.zeros(1)))
        sim.close()
    assert np.isfinite(out[0][2]).all() and out[0][1] > 0.0
    for o in out[1:]:
        assert o[:2] == out[0][:2]
        assert np.array_equal(o[2], out[0][2]) and np.array_equal(o[3], out[0][3])


@pytest.mark.parametrize("recon,precision", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("grid", [(14, 6, 1), (15, 13, 3), (28, 7, 2), (30, 14, 1), (31, 15, 2), (60, 6, 3), (62, 7, 1),
                                  (63, 6, 2), (124, 5, 2), (125, 29, 1), (3, 30, 4), (1, 1, 9)],
                         ids=lambda g: "x".join(map(str, g)))
def test_boxes(lib, grid, recon, precision):
    n1, n2, n3 = grid
    prm = problems.base_problem(n1, n2, n3, recon=recon, precision=precision)
    rng = np.random.default_rng(n1 + n2)
    P0 = np.zeros(problems.params.padded_shape(prm))
    P0[:2] = 1.0 + 0.1 * rng.random(P0[:2].shape)
    P0[2:5] = 0.1 * rng.random(P0[2:5].shape)
    P0[5:] = 0.2 + 0.1 * rng.random(P0[5:].shape)
    same(lib, prm, P0, False)


@pytest.mark.parametrize("recon,precision", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("n1", [14, 28, 30, 62, 63])
def test_bondi_with_electrons_and_radial_clip(lib, n1, recon, precision):
    """the outflow edge's mass flux is that of the last tile's last column"""
    prm, P0 = problems.bondi(n1=n1, n2=14, n3=2, a=0.5, recon=recon, precision=precision)
    prm = dict(prm, bc=[[problems.BC_OUTFLOW, problems.BC_OUTFLOW], *prm["bc"][1:]])
    same(lib, prm, P0, True)


@pytest.mark.parametrize("recon,precision", MODES, ids=MODE_IDS)
def test_cartesian_kerr_schild(lib, recon, precision):
    prm, P0 = problems.cks_bondi(30, 14, 9)
    same(lib, dict(prm, recon=recon, precision=precision), P0, False)


def test_batch_of_narrow_grids(lib):
    jobs = [problems.linear_modes(n=n, n3=9, kvec=(1, 1, 0)) for n in (8, 14, 12)]
    want, dts = [], []
    for prm, P0 in jobs:
        sim = lib.Sim(prm)
        P = sim.to_device(P0)
        dts.append(sim.get_dt(P))
        want.append((sim.run(P, 2, dts[-1]), sim.to_host(P)))
        sim.close()
    for tile in [None] + SHAPES:
        sims = [lib.Sim(prm) for prm, _ in jobs]
        if tile:
            sims[0].set_tiles("sweep", *tile)
        states = [s.to_device(P0) for s, (_, P0) in zip(sims, jobs)]
        b = lib.Batch(sims)
        b.set_dt(dts)
        b.step(states, nsteps=2)
        got, status = b.get()
        assert status == [0, 0, 0] and got == [w[0] for w in want]
        for s, P, w in zip(sims, states, want):
            assert np.array_equal(s.to_host(P), w[1])
        b.close()
        for s in sims:
            s.close()
