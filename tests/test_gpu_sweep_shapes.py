"""The face-flux pass picks its block shape from the grid (one of 512 threads
for grids that fill the chip, 32 x 8 otherwise). Faces on tile seams are computed
by both tiles from the same operands, so the shape changes no bit."""

import numpy as np
import pytest

import problems

pytestmark = pytest.mark.gpu

# grids of more than 1024 large blocks: whole tiles (185 + 1 = 3 x 62, 62 + 1 =
# 9 x 7, 179 + 1 = 6 x 30, 59 + 1 = 4 x 15), one cell more, and ragged ones
GRIDS = [(185, 62, 46), (186, 63, 45), (179, 59, 46), (131, 61, 40)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("recon,precision", [
    (problems.RECON_MC, problems.FP64), (problems.RECON_WENO5, problems.FP64),
    (problems.RECON_MC, problems.MIXED), (problems.RECON_WENO5, problems.MIXED)],
    ids=["mc_fp64", "weno5_fp64", "mc_mixed", "weno5_mixed"])
def test_large_and_small_blocks_give_the_same_bits(lib, grid, recon, precision):
    n1, n2, n3 = grid
    prm, P0 = problems.fm_torus(n1=n1, n2=n2, n3=n3, recon=recon, precision=precision)
    out = []
    for tile in (None, (32, 8)):
        sim = lib.Sim(prm)
        if tile:
            sim.set_tiles("sweep", *tile)
        P, E = sim.to_device(P0), sim.to_device(problems.electron_scalars(P0, prm["gam"]))
        dt = sim.run_electrons(P, E, 2, sim.get_dt(P), "constant", 0.5)
        out.append((dt, sim.to_host(P), sim.to_host(E)))
        sim.close()
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1]) and np.array_equal(out[0][2], out[1][2])
    assert np.isfinite(out[0][1]).all()


def test_cartesian_kerr_schild_shapes(lib):
    prm, P0 = problems.cks_bondi(127, 64, 40)
    out = []
    for tile in (None, (32, 8)):
        sim = lib.Sim(prm)
        if tile:
            sim.set_tiles("sweep", *tile)
        P = sim.to_device(P0)
        dt = sim.run(P, 2, sim.get_dt(P))
        out.append((dt, sim.to_host(P)))
        sim.close()
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])


def test_batch_of_large_blocks_equals_single_contexts(lib):
    jobs = [problems.fm_torus(n1=131, n2=61, n3=30), problems.linear_modes(n=40), problems.bondi(n1=90, n2=33, n3=11, a=0.5)]
    sims = [lib.Sim(prm) for prm, _ in jobs]
    states = [s.to_device(P0) for s, (_, P0) in zip(sims, jobs)]
    dts = [s.get_dt(P) for s, P in zip(sims, states)]
    want = []
    for (prm, P0), dt in zip(jobs, dts):
        sim = lib.Sim(prm)
        P = sim.to_device(P0)
        want.append((sim.run(P, 2, dt), sim.to_host(P)))
        sim.close()
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
