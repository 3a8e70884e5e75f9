"""Synapse-heavy packs whose synapses share reversal potential and decay: a
launch keeps one conductance sum per CV (layout.hpp, kSumMinSteps), shorter
launches and other packs stream every conductance.  Both against the oracle,
with calls of different lengths one after another, so that each path reads
what the other left."""
import numpy as np
import pytest

import oracle
from tests import models
from workloads import gen

TOL = 1e-8  # mV, the parity bar of every register-layout test


def _model(n_branch, n_syn, tau, seed, uniform=True, n_steps=330):
    """Two cells that drive each other: a spike reaches 40 synapses of the
    other cell at 3 delays (several on one CV, some twice), and external events
    hit the soma and random synapses, several in one step."""
    rng = np.random.default_rng(seed)
    cells = []
    for k in range(2):
        d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, n_branch)], rng.integers(3, 9, n_branch),
                             rng.uniform(100, 200, n_branch), rng.uniform(1, 3, n_branch))
        br = rng.integers(n_branch, size=n_syn - 1)
        d.syn = [(-1, 0, tau, 0.0)] + [(int(b), int(rng.integers(d.n_cv[b])), tau, 0.0) for b in br]
        if not uniform:
            d.syn[-1] = d.syn[-1][:2] + (2 * tau, -10.0)
        hit = rng.integers(1, n_syn, size=40)
        d.in_conn = [(1 - k, int(q), int(rng.choice([20, 23, 41])), 2e-4) for q in np.concatenate([hit, hit[:5]])]
        d.ext = [(0, int(s), 0.05) for s in (0, 150)]
        for s in rng.integers(0, n_steps, 12):
            d.ext += [(int(q), int(s), 1e-4) for q in rng.integers(1, n_syn, 9)]
        cells.append(d)
    return gen.assemble(cells, n_steps=n_steps)


# one, two and three groups of entries; a decay that would leave the range of
# doubles within a launch (streamed); synapses that differ (streamed)
CASES = [(64, 12, 800, 2.0, True), (64, 30, 900, 2.0, True), (128, 30, 900, 2.0, True), (256, 30, 900, 2.0, True),
         (64, 20, 800, 1e-3, True), (256, 20, 800, 2.0, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("T,n_branch,n_syn,tau,uniform", CASES)
def test_sums_and_streaming_agree_with_the_oracle(T, n_branch, n_syn, tau, uniform):
    from paper_1901_07454_amd import arbmi
    m = _model(n_branch, n_syn, tau, 5, uniform)
    ref = oracle.Sim(m)
    sim = arbmi.Simulation(m, block_threads=T, coef_mode=3)
    assert sim.info["syn_hbm"] == 1 and sim.info["epoch_steps"] == 20
    done = 0
    for n in (1, 2, 3, 14, 40, 1, 7, 2, 5, 100, 4, 151):
        sim.step(n)
        ref.run(n)
        done += n
        err = np.max(np.abs(sim.voltages_host() - ref.state()["V"]))
        assert err <= TOL, (done, err)
    sp, (g, st, _) = sim.spikes(), ref.spikes()
    assert len(g) >= (2 if tau > 1 else 0)  # the fast synapses never reach threshold
    assert sorted(zip(sp["step"].tolist(), sp["gid"].tolist())) == sorted(zip(st.tolist(), g.tolist()))
    sim.close()


@pytest.mark.gpu
def test_sums_repeat_bit_for_bit():
    """Every CV's sum adds its events in one order: two runs are equal."""
    from paper_1901_07454_amd import arbmi
    m = _model(30, 900, 2.0, 6)
    out = []
    for _ in range(2):
        sim = arbmi.Simulation(m, block_threads=64, coef_mode=3)
        sim.step(330)
        out.append(sim.get_state())
        sim.close()
    assert np.array_equal(out[0], out[1])
