"""The default launch shape (no workgroup size or cells per workgroup asked
for): chosen at the edges of its rule on the CPU (every plan passes the layout
check), and the same results as an explicit shape on the GPU."""
import numpy as np
import pytest

import oracle
from tests import models
from tests.test_abi import _plan
from workloads import gen


def _cells(n, branches, n_cv=8, hh_branches=0):
    out = []
    for _ in range(n):
        d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, branches)] if branches else [], [n_cv] * branches,
                             [150.0] * branches, [2.0] * branches)
        d.mech[:hh_branches] = gen.MECH_HH
        d.gna[:hh_branches], d.gk[:hh_branches], d.gl[:hh_branches] = 0.12, 0.036, 0.0003
        d.syn.append((-1, 0, 2.0, 0.0))
        d.ext.append((0, 3, 0.05))
        out.append(d)
    return out


# (cells, branches, hh branches) -> threads, slots, packs (256 CUs): a cell has branches + 1 tasks
EDGES = [((1, 0, 0), (64, 1, 1)),          # a lone soma
         ((30, 0, 0), (64, 1, 2)),         # 20 hh somas a wave, a thread for every gate
         ((5, 15, 0), (64, 1, 2)),         # 16 tasks: four cells fill a wave
         ((3, 63, 0), (64, 1, 3)),         # 64 tasks: one slot exactly
         ((3, 64, 0), (64, 2, 3)),         # one more: two slots
         ((3, 127, 0), (64, 2, 3)),        # 128 tasks: two slots exactly
         ((3, 128, 0), (256, 1, 3)),       # more than 128 tasks and SIMDs to spare: 256 threads
         ((300, 128, 0), (128, 2, 300)),   # fewer to spare
         ((600, 128, 0), (64, 3, 600)),    # none
         ((3, 255, 0), (256, 1, 3)),
         ((3, 256, 0), (512, 1, 3)),         # more than 256 tasks: two waves per SIMD
         ((3, 511, 0), (512, 1, 3)),
         ((3, 512, 0), (512, 2, 3)),
         ((2, 8, 8), (128, 1, 2)),         # 65 hh CVs
         ((2, 20, 20), (256, 1, 2)),       # 161 hh CVs
         ((1100, 20, 20), (64, 1, 1100))]


@pytest.mark.parametrize("model,shape", EDGES)
def test_shape_at_the_edges(model, shape):
    info = _plan(gen.assemble(_cells(*model[:2], hh_branches=model[2]), n_steps=10))
    assert info["coef_mode"] == 3
    assert (info["block_threads"], info["reg_slots"], info["n_packs"]) == shape


def test_every_size_up_to_the_registers_has_a_plan():
    """Cells that fit 256 threads (up to 768 tasks) take the register layout,
    as with 256 threads asked for, and up to 1024 tasks 512 threads; larger
    ones fall back to streamed coefficients."""
    for nb in list(range(0, 40, 3)) + [126, 127, 128, 191, 192, 383, 384, 511, 512, 766, 767]:
        m = gen.assemble(_cells(1, nb), n_steps=10)
        assert _plan(m)["coef_mode"] == _plan(m, block_threads=256)["coef_mode"] == 3, nb
    assert _plan(gen.assemble(_cells(1, 1023), n_steps=10))["coef_mode"] == 3
    assert _plan(gen.assemble(_cells(1, 1024), n_steps=10))["coef_mode"] == 2


@pytest.mark.gpu
@pytest.mark.parametrize("model", [(3, 0, 0), (9, 15, 0), (2, 64, 0), (2, 128, 0), (2, 8, 8), (3, 20, 20), (2, 256, 30),
                                   (2, 520, 100), (1, 700, 9)])
def test_default_equals_explicit_shape(model):
    """Voltages and spikes of the default shape and of 256 threads with the
    library's packing, the shape used for every model before: the same."""
    from paper_1901_07454_amd import arbmi
    m = gen.assemble(_cells(*model[:2], hh_branches=model[2]), n_steps=300)
    out = []
    for kw in ({}, {"block_threads": 256}):
        sim = arbmi.Simulation(m, **kw)
        sim.step(300)
        out.append((sim.voltages_host(), sim.spikes()))
        sim.close()
    ref = oracle.Sim(m)
    ref.run(300)
    assert np.max(np.abs(out[0][0] - ref.state()["V"])) <= 1e-8
    assert np.max(np.abs(out[0][0] - out[1][0])) <= 1e-8
    assert out[0][1]["step"].tolist() == out[1][1]["step"].tolist()
    assert out[0][1]["gid"].tolist() == out[1][1]["gid"].tolist()


@pytest.mark.gpu
def test_state_blob_of_the_other_default_is_refused():
    """A blob holds the CVs in its layout's order: one from a 256-thread sim
    does not load into a sim whose workgroups the library made smaller, even
    where every size agrees."""
    from paper_1901_07454_amd import arbmi
    m = gen.assemble(_cells(3, 127), n_steps=10)
    a, b = arbmi.Simulation(m), arbmi.Simulation(m, block_threads=256, cells_per_pack=1)
    assert (a.info["n_packs"], a.info["n_slots"]) == (b.info["n_packs"], b.info["n_slots"])
    a.set_state(a.get_state())
    with pytest.raises(arbmi.ArbError):
        a.set_state(b.get_state())
    a.close()
    b.close()


@pytest.mark.gpu
def test_state_blob_of_256_threads_is_refused_by_512():
    """The same for the largest workgroups the library chooses."""
    from paper_1901_07454_amd import arbmi
    m = gen.assemble(_cells(3, 700), n_steps=10)
    a, b = arbmi.Simulation(m), arbmi.Simulation(m, block_threads=256, cells_per_pack=1)
    assert a.info["block_threads"] == 512
    assert (a.info["n_packs"], a.info["n_slots"]) == (b.info["n_packs"], b.info["n_slots"])
    a.set_state(a.get_state())
    with pytest.raises(arbmi.ArbError):
        a.set_state(b.get_state())
    a.close()
    b.close()
