"""Branches longer than the registers under the default shape: cut into
segments of 8 CVs where a cell's segments fit 768 register slots, streamed
otherwise (on the CPU), and against the oracle on the GPU."""
import numpy as np
import pytest

import oracle
from tests import models
from tests.test_abi import _plan
from workloads import gen


def _model(n_cv, parents, hh=(), n_cells=2, n_steps=300, n_syn=1):
    out = []
    for _ in range(n_cells):
        d = models.bare_cell(list(parents), list(n_cv), [3.0 * k for k in n_cv], [2.0] * len(n_cv))
        for b in hh:
            d.mech[b], d.gna[b], d.gk[b], d.gl[b] = gen.MECH_HH, 0.12, 0.036, 0.0003
        d.syn = [(-1, 0, 2.0, 0.0), (len(n_cv) - 1, n_cv[-1] - 1, 1.5, 0.0)] * n_syn
        d.ext += [(0, 3, 0.05), (1, 120, 0.01)]
        out.append(d)
    return gen.assemble(out, n_steps=n_steps)


FAN = (-1, -1, -1, -1, -1)
CASES = [((17,), (-1,), ()), ((24,), (-1,), (0,)), ((25, 16, 17), (-1, 0, 0), (1,)),
         ((100, 1, 8, 9, 33), FAN, (0, 4)),                         # five branches at the soma
         ((31, 40, 23, 7, 64), (-1, -1, 0, 0, 1), range(5)),
         ((700, 3), (-1, 0), ()),                                   # one long chain of segments
         ((700, 600, 760), (-1, 0, 0), ())]                     # more than 256 segments


@pytest.mark.parametrize("n_cv,parents,hh", CASES)
def test_cut_by_default(n_cv, parents, hh):
    m = _model(n_cv, parents, hh)
    info, streamed = _plan(m), _plan(m, coef_mode=2)
    assert info["coef_mode"] == streamed["coef_mode"] == 2
    assert info["reg_slots"] > 0 and info["reg_len"] == 8 and info["syn_hbm"] == 0
    assert streamed["reg_slots"] == 0


def test_streamed_where_asked_for_or_too_large():
    from paper_1901_07454_amd import arbmi
    m = _model((100, 30), (-1, 0))
    for kw in ({"block_threads": 256}, {"cells_per_pack": 1}, {"flags": arbmi.ARB_FLAG_GRADIENTS}):
        info = _plan(m, **kw)
        assert info["coef_mode"] == 2 and info["reg_slots"] == 0, kw
    # too many segments; LDS for the forward pass, not for the adjoint
    for n_cv in ((7000,), (4000,)):
        info = _plan(_model(n_cv, (-1,), n_cells=1))
        assert info["coef_mode"] == 2 and info["reg_slots"] == 0, n_cv
    # more synapses than the registers' layout keeps in LDS
    assert _plan(_model((100, 30), (-1, 0), n_syn=400))["reg_slots"] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("n_cv,parents,hh", CASES)
def test_cut_matches_oracle(n_cv, parents, hh):
    """Voltages and spikes to the tolerance of the other layouts' tests."""
    from paper_1901_07454_amd import arbmi
    m = _model(n_cv, parents, hh)
    ref = oracle.Sim(m)
    ref.run(300)
    for kw in ({}, {"flags": arbmi.ARB_FLAG_GRAPH}):
        sim = arbmi.Simulation(m, **kw)
        assert sim.info["reg_slots"] > 0
        sim.step(300)
        V, sp = sim.voltages_host(), sim.spikes()
        sim.close()
        assert np.max(np.abs(V - ref.state()["V"])) <= 1e-8
        gid, step, _ = ref.spikes()
        assert sp["step"].tolist() == step.tolist() and sp["gid"].tolist() == gid.tolist()


@pytest.mark.gpu
def test_gradients_without_the_flag():
    """A sim built without the gradient flag still takes gradient calls, after
    ordinary steps too, and agrees with the oracle's adjoint as the streamed
    layout does (1e-7 relative)."""
    import torch

    from paper_1901_07454_amd import arbmi
    from tests.test_gpu_adjoint import model_theta
    n = 300
    m = _model((33, 17, 24), (-1, 0, 0), hh=(1,))
    th = model_theta(m)
    sim = arbmi.Simulation(m)
    assert sim.info["reg_slots"] > 0
    state0 = sim.get_state()
    sim.step(20)
    sim.set_state(state0)
    trace = torch.empty(2, n, dtype=torch.float64, device="cuda")
    arbmi.arb_grad_forward(sim.h, n, 50, trace)
    tr = trace.cpu().numpy()
    dl = np.cos(0.01 * np.arange(tr.size)).reshape(tr.shape) / tr.size
    out = torch.empty(th.size, dtype=torch.float64, device="cuda")
    arbmi.arb_grad_backward(sim.h, torch.as_tensor(dl, device="cuda"), out)
    g = out.cpu().numpy().reshape(-1, 3)
    sim.close()
    otr, og = oracle.Sim(m).adjoint(n, dl)
    assert np.max(np.abs(tr - otr)) <= 1e-8
    den = np.maximum(np.abs(og), 1e-3 * np.max(np.abs(og), axis=0, keepdims=True))
    assert (np.abs(g - og) / den).max() <= 1e-7


@pytest.mark.gpu
def test_blob_of_the_streamed_layout_is_refused():
    from paper_1901_07454_amd import arbmi
    m = _model((24, 24), (-1, 0))
    a, b = arbmi.Simulation(m), arbmi.Simulation(m, coef_mode=2)
    a.step(20)
    a.set_state(a.get_state())
    with pytest.raises(arbmi.ArbError):
        a.set_state(b.get_state())
    a.close()
    b.close()
