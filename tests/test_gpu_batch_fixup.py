"""The fixup of a batch gives each job a fixed number of blocks, which stride over
its tiles (682 a job for three jobs, 64 for forty): failed zones in the first,
a middle and the last tiles of every job end as in a context of their own."""

import numpy as np
import pytest

import problems

pytestmark = pytest.mark.gpu
NG = 3


def spoil(prm, P0):
    P0 = P0.copy()
    for k, j, i in ((0, 0, 0), (prm["n3"] // 2, prm["n2"] // 2, prm["n1"] // 2),
                    (prm["n3"] - 1, prm["n2"] - 1, prm["n1"] - 1)):
        P0[1, NG + k, NG + j, NG + i] = np.nan
    return prm, P0


@pytest.mark.parametrize("make", [
    lambda: [problems.linear_modes(n=6), problems.fm_torus(n1=96, n2=64, n3=40), problems.linear_modes(n=32)],
    lambda: [problems.linear_modes(n=16) for _ in range(40)],
], ids=["3_jobs", "40_jobs"])
def test_failed_zones_of_a_batch_are_repaired_as_in_single_contexts(lib, make):
    clean = make()
    sims = [lib.Sim(prm) for prm, _ in clean]
    dts = [s.get_dt(s.to_device(P0)) for s, (_, P0) in zip(sims, clean)]
    jobs = [spoil(*job) for job in clean]
    want = []
    for s, (_, P0), dt in zip(sims, jobs, dts):
        P = s.to_device(P0)
        dt = s.run(P, 1, dt)
        assert s.step_failures() > 0
        want.append((dt, s.to_host(P)))
    states = [s.to_device(P0) for s, (_, P0) in zip(sims, jobs)]
    batch = lib.Batch(sims)
    batch.set_dt(dts)
    batch.step(states, nsteps=1)
    got_dt, status = batch.get()
    batch.close()
    for s, (prm, _), P, (dt, ref), d in zip(sims, jobs, states, want, got_dt):
        got = s.to_host(P)
        assert d == dt and np.array_equal(got, ref, equal_nan=True)  # ghosts still hold the spoiled values
        assert np.isfinite(got[:, NG:NG + prm["n3"], NG:NG + prm["n2"], NG:NG + prm["n1"]]).all()
        s.close()
    assert not any(status)
