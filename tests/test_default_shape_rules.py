"""The default launch shape's rules that count workgroups on a CU: plans on the
CPU, results against the oracle on the GPU."""
import numpy as np
import pytest

import oracle
from paper_1901_07454_amd import arbmi
from tests.test_abi import _plan
from tests.test_default_shape import _cells
from workloads import gen


def _shape(cells, **kw):
    info = _plan(gen.assemble(cells, n_steps=10), **kw)
    return info["block_threads"], info["reg_slots"], info["n_packs"]


@pytest.mark.parametrize("n,branches,hh,shape", [
    (256, 300, 0, (512, 1, 256)),   # a CU for each cell
    (257, 300, 30, (256, 2, 257)),  # two of 62 KB share one
    (300, 400, 17, (256, 2, 300)),  # 70 KB
    (300, 380, 95, (512, 1, 300))])  # 110 KB: one to a CU either way
def test_512_threads_where_a_cell_has_a_cu(n, branches, hh, shape):
    assert _shape(_cells(1, branches, hh_branches=hh) * n) == shape


@pytest.mark.parametrize("branches,n_syn,same,shape", [
    (130, 700, True, (64, 3, 600)),     # one conductance sum per CV
    (130, 700, False, (256, 1, 600)),   # streamed: a thread for every branch
    (63, 700, False, (64, 1, 600))])    # one wave has them
def test_threads_for_streamed_synapses(branches, n_syn, same, shape):
    d = _cells(1, branches)[0]
    d.syn = [(-1, 0, 2.0, 0.0)] + [(q % branches, 0, 2.0 if same or q % 2 else 3.0, 0.0) for q in range(n_syn - 1)]
    assert _shape([d] * 600) == shape


def _mixed(n, big, seed=3):
    """n cells of 3 to 60 branches and one of `big`."""
    rng = np.random.default_rng(seed)
    out = [_cells(1, big, hh_branches=big // 8)[0]]
    for nb in rng.integers(3, 60, n - 1):
        out.append(_cells(1, int(nb), hh_branches=int(nb) // 8)[0])
    return out


def test_mixed_cells_share_workgroups():
    T, _, packs = _shape(_mixed(600, 230))
    assert T == 256 and 200 <= packs <= 256
    T, _, packs = _shape(_mixed(200, 230))  # a CU for each
    assert T == 256 and packs == 200


@pytest.mark.gpu
@pytest.mark.parametrize("n,big", [(300, 230), (300, 383)])
def test_mixed_cells_match_the_oracle(n, big):
    m = gen.assemble(_mixed(n, big), n_steps=60)
    ref = oracle.Sim(m)
    ref.run(60)
    sim = arbmi.Simulation(m)
    assert sim.info["block_threads"] >= 256 and sim.info["n_packs"] <= 256
    sim.step(30)
    blob = sim.get_state()
    sim.step(30)
    V = sim.voltages_host()
    assert np.max(np.abs(V - ref.state()["V"])) <= 1e-8
    sim.set_state(blob)
    sim.step(30)
    assert np.array_equal(sim.voltages_host(), V)
    sim.close()
