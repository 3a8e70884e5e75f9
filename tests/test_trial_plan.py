"""The autotuner times the library's own launch shape as the full model will
have it, though on a sample of its cells (host build of the planner)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_own_shape_is_the_full_models(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "plan_check")
    subprocess.run(["hipcc", "-O1", "-std=c++17", "-o", exe, os.path.join(HERE, "plan_check.cpp"),
                    os.path.join(HERE, "..", "paper_1901_07454_amd", "csrc", "plan.cpp")],
                   check=True, capture_output=True, timeout=600)

    def plans(*args):
        out = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True, timeout=60).stdout
        return [tuple(map(int, line.split())) for line in out.split("\n") if line]

    # 100 synapses a cell: 128 threads where SIMDs are idle, one wave otherwise
    full, sample, own, explicit = plans(3000, 160, 100)
    assert full != sample and (full[1], sample[1]) == (64, 128)
    assert own == full
    assert explicit[:2] == (3, 128)
    # where the rules see no difference, neither does the trial
    full, sample, own, _ = plans(100, 100, 100)
    assert own == full == sample
