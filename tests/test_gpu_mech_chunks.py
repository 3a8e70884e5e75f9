"""Generated mechanisms: the order in which a pack's instances are advanced."""
import numpy as np
import pytest

import oracle
from tests import models
from workloads import gen

pytestmark = pytest.mark.gpu
TOL = 1e-8  # mV, the suite's parity bar


@pytest.mark.parametrize("T,n_hh_branches", [(64, 8), (64, 9), (256, 16), (256, 17)])
def test_chunks_of_instances_at_their_edges(T, n_hh_branches):
    """Instances are advanced in chunks of 128 of one mechanism, two to a
    lane, or one where the chunk's second half is empty: hh_dsl on 64 or 72
    CVs (half a chunk and one branch more) or 128 and 136 (a whole one and
    more), kdr on the rest, hcn alone in its chunk, against the oracle; calls
    of different lengths agree bit for bit."""
    from paper_1901_07454_amd import arbmi
    nb = 40
    d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, nb)], [8] * nb, [150.0] * nb, [2.0] * nb)
    d.syn.append((-1, 0, 2.0, 0.0))
    d.ext += [(0, 5, 0.05), (0, 300, 0.05)]
    dens = [(0, -1, "hcn", {"gbar": 3e-4})]
    dens += [(0, b, "hh_dsl", {"gnabar": 0.04, "gkbar": 0.012}) for b in range(n_hh_branches)]
    dens += [(0, b, "kdr", {"gbar": 2e-3}) for b in range(n_hh_branches, nb)]
    m = gen.with_densities(gen.assemble([d], n_steps=500), dens)
    ref = oracle.Sim(m)
    ref.run(500)
    out = []
    for calls in ((500,), (1, 2, 97, 400)):
        sim = arbmi.Simulation(m, block_threads=T)
        for n in calls:
            sim.step(n)
        out.append(sim.voltages_host())
        sim.close()
    assert np.max(np.abs(out[0] - ref.state()["V"])) <= TOL
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("nb,T", [(31, 256), (32, 512), (70, 512)])
def test_default_threads(nb, T):
    """The library's choice: 512 threads from 257 CVs on; results as the oracle's."""
    from paper_1901_07454_amd import arbmi
    d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, nb)], [8] * nb, [150.0] * nb, [2.0] * nb)
    d.syn.append((-1, 0, 2.0, 0.0))
    d.ext += [(0, 5, 0.05), (0, 200, 0.05)]
    dens = [(0, b, "hh_dsl", {"gnabar": 0.04, "gkbar": 0.012}) for b in range(nb // 2)]
    dens += [(0, b, "kdr", {"gbar": 2e-3}) for b in range(nb // 3, nb)]
    m = gen.with_densities(gen.assemble([d], n_steps=300), dens)
    ref = oracle.Sim(m)
    ref.run(300)
    sim = arbmi.Simulation(m)
    assert sim.info["block_threads"] == T
    sim.step(300)
    V = sim.voltages_host()
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= TOL
