"""Generated mechanisms: where a launch keeps the instances' currents (LDS, or
HBM where LDS has no room or would hold too few workgroups), against the
oracle."""
import numpy as np
import pytest

import oracle
from tests import models
from workloads import gen

pytestmark = pytest.mark.gpu
TOL = 1e-8  # mV, the suite's parity bar


def _cell(nb, n_cv=8):
    d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, nb)], [n_cv] * nb, [150.0] * nb, [2.0] * nb)
    d.syn.append((-1, 0, 2.0, 0.0))
    d.ext += [(0, 5, 0.05), (0, 120, 0.05)]
    return d


def _dens(c, nb, kinds):
    out = [(c, -1, "hcn", {"gbar": 3e-4})]
    for k in range(kinds):
        out += [(c, b, ("kdr", "hh_dsl", "hcn", "kdr")[k], {("gbar", "gnabar", "gbar", "gbar")[k]: 1e-3})
                for b in range(k, nb)]
    return out


@pytest.mark.parametrize("T,nb,kinds", [(0, 300, 1), (0, 300, 4), (256, 300, 4), (0, 360, 4), (256, 360, 4)])
def test_one_large_cell(T, nb, kinds):
    """2401 and 2881 CVs with up to four instances each: their currents fit
    LDS beside the cell, or do not."""
    from paper_1901_07454_amd import arbmi
    m = gen.with_densities(gen.assemble([_cell(nb)], n_steps=150), _dens(0, nb, kinds))
    ref = oracle.Sim(m)
    ref.run(150)
    out = []
    for calls in ((150,), (1, 49, 100)):
        sim = arbmi.Simulation(m, block_threads=T)
        for n in calls:
            sim.step(n)
        out.append(sim.voltages_host())
        sim.close()
    assert np.max(np.abs(out[0] - ref.state()["V"])) <= TOL
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("T,n_cells,nb", [(256, 2600, 31), (128, 2600, 31), (64, 1500, 15), (0, 600, 7), (0, 2100, 15)])
def test_many_cells(T, n_cells, nb):
    """Equal cells filling workgroups of several, more of these than CUs take
    at once: every cell as the oracle's one."""
    from paper_1901_07454_amd import arbmi
    one = gen.with_densities(gen.assemble([_cell(nb)], n_steps=150), _dens(0, nb, 2))
    ref = oracle.Sim(one)
    ref.run(150)
    m = gen.with_densities(gen.assemble([_cell(nb)] * n_cells, n_steps=150),
                           [e for c in range(n_cells) for e in _dens(c, nb, 2)])
    sim = arbmi.Simulation(m, block_threads=T)
    sim.step(150)
    V = sim.voltages_host().reshape(n_cells, -1)
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= TOL
