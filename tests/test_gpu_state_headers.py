"""Saved states and the default launch shape: a blob of 256 threads filled with
cells (what the default was, and an explicit 256 threads is) loads where the
default packs the same cells the same way, and nowhere else."""
import numpy as np
import pytest

from tests import models
from workloads import gen

pytestmark = pytest.mark.gpu


def _model(n_branch, n_syn):
    cells = []
    for k, nb in enumerate(n_branch):
        d = models.bare_cell([-1] + [(b - 1) // 2 for b in range(1, nb)], [8] * nb, [150.0] * nb, [2.0] * nb)
        d.syn = [(-1, 0, 2.0, 0.0)] + [(q % 36, q % 8, 2.0, 0.0) for q in range(n_syn - 1)]
        d.ext = [(0, 3, 0.05)] if k == 0 else []  # in the first workgroup either way
        cells.append(d)
    return gen.assemble(cells, n_steps=60)


# the largest cell asks for 256 threads; the others go six to a workgroup by
# LDS, fewer by the default's rule (two workgroups either way), or one each
CASES = [((130,) + (60,) * 5, 63, False), ((130,) + (44,) * 6, 63, False), ((130,) + (70,) * 4, 80, False),
         ((255,), 3, True), ((250, 240, 230), 300, True)]


@pytest.mark.parametrize("n_branch,n_syn,same", CASES)
def test_blob_of_256_threads_loads_where_the_layout_is_the_same(n_branch, n_syn, same):
    from paper_1901_07454_amd import arbmi
    m = _model(n_branch, n_syn)
    a, b = arbmi.Simulation(m), arbmi.Simulation(m, block_threads=256)
    assert a.info["block_threads"] == 256 and not (same and a.info["n_packs"] != b.info["n_packs"])
    assert (a.info["n_packs"], a.info["n_slots"]) == (b.info["n_packs"], b.info["n_slots"])
    b.step(20)
    blob = b.get_state()
    if same:
        a.set_state(blob)
        assert np.array_equal(a.voltages_host(), b.voltages_host())
    else:
        with pytest.raises(arbmi.ArbError):
            a.set_state(blob)
    a.step(20)
    own, V = a.get_state(), a.voltages_host()
    a.step(20)
    a.set_state(own)
    assert np.array_equal(a.voltages_host(), V)
    a.close()
    b.close()
