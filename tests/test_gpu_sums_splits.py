"""Synapse-heavy packs that carry conductance sums: the sums are state, so
results are the same bit for bit however a run is split into calls, launches
and epochs, and through a saved state; and 512 threads, which take two CVs at a
time, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_synapse_sums import TOL, _model

pytestmark = pytest.mark.gpu
N = 330


def _cells_state(blob):
    """The part of a saved state that the cells' equations hold: voltages, gates
    and conductances (the rest has event and spike buffers, whose unused places
    are arbitrary), and the blob's last value, the last pack's decay since its
    conductances were exact."""
    raw = bytes(blob)
    _, _, n_slots, n_hh, n_syn = np.frombuffer(raw, np.int64, 5)
    return raw[80:80 + 8 * int(n_slots + 3 * n_hh + n_syn)] + raw[-8:]


def _run(m, calls, **kw):
    from paper_1901_07454_amd import arbmi
    sim = arbmi.Simulation(m, coef_mode=3, **kw)
    assert sim.info["syn_hbm"] == 1
    for n in calls:
        sim.step(n)
    out = sim.voltages_host(), sim.spikes(), _cells_state(sim.get_state())
    sim.close()
    return out


# one, two and three groups of entries; a decay of 0.43 a step, whose
# conductances are scaled every 110 steps; synapses that differ (streamed)
CASES = [(64, 12, 800, 2.0, True), (64, 30, 900, 2.0, True), (128, 30, 900, 2.0, True), (256, 30, 900, 0.03, True),
         (64, 20, 800, 2.0, False)]


@pytest.mark.parametrize("T,n_branch,n_syn,tau,uniform", CASES)
def test_splits_agree_bit_for_bit(T, n_branch, n_syn, tau, uniform):
    from paper_1901_07454_amd import arbmi
    m = _model(n_branch, n_syn, tau, 5, uniform, n_steps=N)
    V, sp, state = _run(m, (N,), block_threads=T)
    for calls, kw in (((1,) * N, {}), ((1, 2, 3, 14, 40, 1, 7, 2, 5, 100, 4, 151), {}), ((N,), {"epoch_steps": 1}),
                      ((165, 165), {"epoch_steps": 7}), ((N,), {"flags": arbmi.ARB_FLAG_GRAPH})):
        v, s, b = _run(m, calls, block_threads=T, **kw)
        assert np.array_equal(V, v), (calls, kw)
        assert np.array_equal(sp, s), (calls, kw)
        n = len(state) - (0 if uniform else 8)
        assert state[:n] == b[:n], (calls, kw)


@pytest.mark.parametrize("at", [1, 105, 170])
def test_saved_state_continues_bit_for_bit(at):
    """n steps, a saved state and the rest in another sim: as in one run, at
    an epoch's first step, between two, and after a scaling (decay 0.43)."""
    from paper_1901_07454_amd import arbmi
    m = _model(30, 900, 0.03, 6, n_steps=N)
    V, sp, state = _run(m, (N,), block_threads=128)
    a, b = (arbmi.Simulation(m, block_threads=128, coef_mode=3) for _ in range(2))
    a.step(at)
    s1 = a.spikes()
    b.set_state(a.get_state())
    b.step(N - at)
    assert np.array_equal(b.voltages_host(), V)
    assert np.array_equal(np.concatenate([s1, b.spikes()]), sp)
    assert _cells_state(b.get_state()) == state
    a.close()
    b.close()


@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("n_branch", [260, 520])
def test_512_threads_match_the_oracle(n_branch, uniform):
    """Cells of more than 256 branches by default: two entries at a time, more
    entries than threads (an odd number of groups or the second entry absent),
    sums and streaming, calls of different lengths."""
    from paper_1901_07454_amd import arbmi
    m = _model(n_branch, 900, 2.0, 8, uniform, n_steps=N)
    ref = oracle.Sim(m)
    sim = arbmi.Simulation(m)
    assert sim.info["block_threads"] == 512 and sim.info["syn_hbm"] == 1
    for n in (1, 2, 3, 14, 40, 1, 7, 2, 5, 100, 4, 151):
        sim.step(n)
        ref.run(n)
        assert np.max(np.abs(sim.voltages_host() - ref.state()["V"])) <= TOL
    gid, step, _ = ref.spikes()
    sp = sim.spikes()
    assert sp["step"].tolist() == step.tolist() and sp["gid"].tolist() == gid.tolist()
    sim.close()


@pytest.mark.parametrize("T", [64, 256])
def test_both_kinds_in_one_launch(T):
    """Cells that carry sums, cells that stream and a cell with its synapses
    in LDS, in one launch class (the variant for sums), against the oracle."""
    from paper_1901_07454_amd import arbmi
    from tests import models
    from workloads import gen
    rng = np.random.default_rng(3)
    cells = []
    for n_syn, tau2 in ((800, 2.0), (800, 3.0), (20, 2.0), (900, 2.0)):
        d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, 40)], rng.integers(3, 9, 40),
                             rng.uniform(100, 200, 40), rng.uniform(1, 3, 40))
        br = rng.integers(40, size=n_syn - 1)
        d.syn = [(-1, 0, 2.0, 0.0)] + [(int(b), int(rng.integers(d.n_cv[b])), 2.0, 0.0) for b in br]
        d.syn[-1] = d.syn[-1][:2] + (tau2, 0.0)
        d.ext = [(0, 3, 0.05)] + [(int(q), int(s), 1e-3) for q, s in zip(rng.integers(n_syn, size=200),
                                                                         rng.integers(0, 200, 200))]
        cells.append(d)
    m = gen.assemble(cells, n_steps=200)
    ref = oracle.Sim(m)
    ref.run(200)
    sim = arbmi.Simulation(m, block_threads=T, coef_mode=3, cells_per_pack=1)
    assert sim.info["n_packs"] == 4 and sim.info["n_classes"] == 1
    sim.step(200)
    V = sim.voltages_host()
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= TOL
