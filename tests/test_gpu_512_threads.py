"""Workgroups of 512 threads (the library's choice for cells of more than 256
branches) whose state is held in HBM."""
import numpy as np
import pytest

import oracle
from tests import models
from workloads import gen

pytestmark = pytest.mark.gpu
TOL = 1e-8  # mV, the parity bar of every register-layout test


def test_no_hh_instance():
    """A passive cell of 900 CVs with synapses, too large for LDS with its
    nonlinear CVs' constants: they are read from HBM, and conductances of hh
    instances, of which there are none, are not."""
    from paper_1901_07454_amd import arbmi
    nb = 960
    cells = []
    for _ in range(2):
        d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, nb)], [8] * nb, [150.0] * nb, [2.0] * nb,
                             soma_mech=gen.MECH_PAS)
        d.syn = [(-1, 0, 2.0, 0.0)] + [(q, q % 8, 2.0 + (q % 2), 0.0) for q in range(900)]
        d.ext = [(q, q % 50, 1e-3) for q in range(0, 901, 7)]
        cells.append(d)
    m = gen.assemble(cells, n_steps=100)
    ref = oracle.Sim(m)
    ref.run(100)
    sim = arbmi.Simulation(m)
    assert sim.info["block_threads"] == 512 and sim.info["syn_hbm"] == 1 and sim.info["n_hh"] == 0
    sim.step(100)
    V = sim.voltages_host()
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= TOL
