"""The default launch shape of many similar cells, where the estimated step
decides: plans on the CPU, and results as the oracle's on the GPU."""
import numpy as np
import pytest

import oracle
from tests.test_abi import _plan
from tests.test_default_shape import _cells
from workloads import gen


def _model(n, branches, n_cv, hh):
    return gen.assemble(_cells(1, branches, n_cv, hh) * n, n_steps=60)


# (cells, branches, CVs, hh branches) -> threads, workgroups (256 CUs)
@pytest.mark.parametrize("model,shape", [((1500, 20, 13, 0), (64, 500)),    # three cells a wave: one round of waves
                                         ((300, 20, 13, 0), (64, 300)),     # a round either way: by rule
                                         ((5152, 15, 8, 8), (256, 736)),    # seven cells of 65 hh CVs
                                         ((600, 63, 13, 6), (256, 200)),    # three of 64 branches, one to a thread
                                         ((255, 63, 13, 6), (128, 255)),    # fewer cells than CUs: by rule
                                         ((1537, 63, 8, 0), (64, 1537))])
def test_shape(model, shape):
    info = _plan(_model(*model))
    assert (info["block_threads"], info["n_packs"]) == shape
    assert info["lds_bytes"] <= (160 * 1024 - 256) // 2


@pytest.mark.gpu
@pytest.mark.parametrize("n,branches,n_cv,hh", [(1500, 20, 13, 0), (1400, 15, 8, 8), (600, 63, 13, 6), (2600, 3, 13, 1)])
def test_every_cell_as_the_oracle(n, branches, n_cv, hh):
    from paper_1901_07454_amd import arbmi
    ref = oracle.Sim(_model(1, branches, n_cv, hh))
    ref.run(60)
    sim = arbmi.Simulation(_model(n, branches, n_cv, hh))
    sim.step(40)
    blob = sim.get_state()
    sim.step(20)
    V = sim.voltages_host().reshape(n, -1)
    assert np.max(np.abs(V - ref.state()["V"])) <= 1e-8
    sim.set_state(blob)
    sim.step(20)
    assert np.array_equal(sim.voltages_host().reshape(n, -1), V)
    sim.close()
