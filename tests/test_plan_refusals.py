"""Layouts that are asked for and cannot be had are refused, with the reason
(CPU: plans only)."""
import ctypes as C

import pytest

from paper_1901_07454_amd import arbmi
from tests.test_abi import _plan
from tests.test_default_shape import _cells
from workloads import gen


@pytest.mark.parametrize("branches,fits", [(767, True), (768, False), (1023, False)])
def test_register_layout_asked_for_takes_768_branches(branches, fits):
    """256 threads hold three branches each, the soma's among them; without a
    request the library may take 512 threads for more."""
    m = gen.assemble(_cells(1, branches), n_steps=10)
    for kw in ({}, {"block_threads": 256}):
        if fits:
            assert _plan(m, coef_mode=3, **kw)["coef_mode"] == 3
        else:
            with pytest.raises(arbmi.ArbError, match="register"):
                _plan(m, coef_mode=3, **kw)
    assert _plan(m)["coef_mode"] == 3


def test_generated_mechanisms_on_long_branches():
    """Branches of more than 16 CVs with generated mechanisms: the plan is
    refused with what to ask for, and what was asked for is planned."""
    m = gen.assemble(_cells(1, 40, 24), n_steps=10)
    dens = arbmi.density_structs([(0, b, "kdr", {}) for b in range(40)])
    kw = {"densities": C.cast(dens, C.c_void_p), "n_densities": len(dens)}
    with pytest.raises(arbmi.ArbError, match="coef_mode 3"):
        _plan(m, **kw)
    info = _plan(m, coef_mode=3, **kw)
    assert info["coef_mode"] == 3 and info["reg_len"] == 8 and info["reg_slots"] > 0
