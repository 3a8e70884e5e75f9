"""The default launch shape of many small cells with generated mechanisms:
several to a workgroup of 256 threads (plans on the CPU), and the same results
as the oracle's."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_1901_07454_amd import arbmi
from tests.test_abi import _plan
from tests.test_gpu_mech_currents import TOL, _cell, _dens
from workloads import gen


def _planned(n, nb, n_syn=1):
    dens = arbmi.density_structs([e for c in range(n) for e in _dens(c, nb, 1)])
    d = _cell(nb)
    d.syn = d.syn * n_syn
    info = _plan(gen.assemble([d] * n, n_steps=10), densities=C.cast(dens, C.c_void_p), n_densities=len(dens))
    return info["block_threads"], info["n_packs"]


# (cells, branches) -> threads, workgroups (256 CUs): a cell has 8 branches + 1 CVs
@pytest.mark.parametrize("n,nb,shape", [(511, 7, (64, 511)), (512, 7, (256, 256)), (1100, 7, (256, 275)),
                                        (6000, 7, (256, 353)),     # 1024 // 57 = 17 cells
                                        (600, 31, (256, 300)), (1300, 31, (256, 325)),  # at most 4 of 249 CVs
                                        (600, 63, (256, 300)),     # two of 505
                                        (600, 127, (256, 600))])   # one of 1017
def test_cells_share_256_threads(n, nb, shape):
    assert _planned(n, nb) == shape


@pytest.mark.parametrize("n_syn,packs", [(85, 263), (86, 300), (170, 525), (341, 1050), (342, 2100), (682, 2100)])
def test_shared_synapses_stay_in_lds(n_syn, packs):
    """At most 682 synapses to a workgroup: more would be kept in HBM, which
    cells with generated mechanisms are refused for."""
    assert _planned(2100, 15, n_syn)[1] == packs


@pytest.mark.gpu
@pytest.mark.parametrize("n,nb", [(512, 7), (700, 15), (520, 63)])
def test_shared_threads_match_the_oracle(n, nb):
    one = gen.with_densities(gen.assemble([_cell(nb)], n_steps=150), _dens(0, nb, 2))
    ref = oracle.Sim(one)
    ref.run(150)
    m = gen.with_densities(gen.assemble([_cell(nb)] * n, n_steps=150), [e for c in range(n) for e in _dens(c, nb, 2)])
    sim = arbmi.Simulation(m)
    assert sim.info["block_threads"] == 256 and sim.info["n_packs"] < n
    sim.step(150)
    V = sim.voltages_host().reshape(n, -1)
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= TOL
