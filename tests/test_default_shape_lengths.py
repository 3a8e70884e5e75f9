"""The default launch shape for branches of 9 to 16 CVs, of which a thread
holds one: cells of more than 256 branches have no register layout (streamed by
default, refused where the register layout is asked for), and every plan is one
that has a kernel."""
import numpy as np
import pytest

import oracle
from paper_1901_07454_amd import arbmi
from tests.test_abi import _plan
from tests.test_default_shape import _cells
from workloads import gen


@pytest.mark.parametrize("branches", [1, 63, 64, 128, 255, 256, 300, 400, 511, 512, 700, 1023, 1024])
@pytest.mark.parametrize("n_cv", [8, 9, 10, 12, 16, 17])
def test_every_plan_has_a_kernel(branches, n_cv):
    for n, kw in ((1, {}), (300, {}), (1, {"flags": arbmi.ARB_FLAG_GRADIENTS})):
        if n > 1 and branches > 300:
            continue
        cells = _cells(1, branches, n_cv)
        m = gen.assemble(cells * n, n_steps=10)
        try:
            info = _plan(m, **kw)
        except arbmi.ArbError:  # too large for a CU's LDS: streamed coefficients do not fit either
            with pytest.raises(arbmi.ArbError, match="LDS"):
                _plan(m, coef_mode=2, **kw)
            continue
        T, S, L = info["block_threads"], info["reg_slots"], info["reg_len"]
        if 8 < n_cv <= 16:
            # one branch a thread, at most 256 of them, the soma's among them
            assert info["coef_mode"] == (3 if branches < 256 and not (kw and S == 0) else 2)
        if S == 0:
            assert info["coef_mode"] == 2
            continue
        assert (L, S) in ((8, 1), (8, 2), (8, 3), (16, 1))
        assert T in (64, 128, 256) or (T == 512 and L == 8 and S <= 2 and not kw)


def test_refused_where_asked_for():
    m = gen.assemble(_cells(1, 300, 12), n_steps=10)
    with pytest.raises(arbmi.ArbError, match="register"):
        _plan(m, coef_mode=3)
    assert _plan(gen.assemble(_cells(1, 255, 12), n_steps=10), coef_mode=3)["coef_mode"] == 3


@pytest.mark.gpu
@pytest.mark.parametrize("branches,n_cv", [(255, 16), (256, 9), (300, 12), (511, 16)])
def test_steps_as_the_oracle(branches, n_cv):
    """One such cell, alone and beside a small one, to the suite's 1e-8 mV."""
    for cells in (_cells(1, branches, n_cv), _cells(1, branches, n_cv) + _cells(2, 3, 8)):
        m = gen.assemble(cells, n_steps=200)
        ref = oracle.Sim(m)
        ref.run(200)
        sim = arbmi.Simulation(m)
        sim.step(200)
        V, sp = sim.voltages_host(), sim.spikes()
        sim.close()
        assert np.max(np.abs(V - ref.state()["V"])) <= 1e-8
        gid, step, _ = ref.spikes()
        assert sp["step"].tolist() == step.tolist() and sp["gid"].tolist() == gid.tolist()
