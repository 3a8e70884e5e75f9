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


GRADS = {"flags": arbmi.ARB_FLAG_GRADIENTS}


@pytest.mark.parametrize("n,branches,n_cv,hh,T", [
    (800, 25, 8, 25, 256),    # three to 256 threads leave more than two thirds of the CUs one
    (120, 15, 8, 1, 64),      # they would not
    (30, 50, 13, 0, 256), (30, 30, 13, 0, 64)])  # more than 40 branches of up to 16 CVs
def test_threads_for_gradients(n, branches, n_cv, hh, T):
    assert _shape(_cells(1, branches, n_cv, hh) * n, **GRADS)[0] == T


@pytest.mark.gpu
@pytest.mark.parametrize("n,branches,n_cv,hh", [(600, 25, 8, 25), (20, 50, 13, 0)])
def test_gradients_match_the_oracle(n, branches, n_cv, hh):
    """Every cell's trace and gradient as the oracle's for one cell: 1e-8 mV
    and 1e-7 relative, the bounds of the other layouts' tests."""
    import torch

    from tests.test_gpu_adjoint import model_theta
    steps = 120
    one = gen.assemble(_cells(1, branches, n_cv, hh), n_steps=steps)
    m = gen.assemble(_cells(1, branches, n_cv, hh) * n, n_steps=steps)
    sim = arbmi.Simulation(m, **GRADS)
    assert sim.info["block_threads"] == 256 and sim.info["coef_mode"] == 3
    trace = torch.empty(n, steps, dtype=torch.float64, device="cuda")
    arbmi.arb_grad_forward(sim.h, steps, 50, trace)
    dl = np.cos(0.05 * np.arange(steps))[None, :] / steps
    out = torch.empty(n * model_theta(one).size, dtype=torch.float64, device="cuda")
    arbmi.arb_grad_backward(sim.h, torch.as_tensor(np.repeat(dl, n, axis=0), device="cuda"), out)
    tr, g = trace.cpu().numpy(), out.cpu().numpy().reshape(n, -1, 3)
    sim.close()
    otr, og = oracle.Sim(one).adjoint(steps, dl)
    assert np.max(np.abs(tr - otr)) <= 1e-8
    den = np.maximum(np.abs(og), 1e-3 * np.max(np.abs(og), axis=0, keepdims=True))
    assert (np.abs(g - og.reshape(1, -1, 3)) <= 1e-7 * den.reshape(1, -1, 3)).all()  # (no passive region: 0 <= 0)
