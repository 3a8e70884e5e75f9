"""Generated mechanisms far outside the physiological range: exponentials that
overflow or vanish saturate as the described arithmetic does (a gate whose
midpoint lies far away is closed, not undefined)."""
import subprocess

import numpy as np
import pytest

import oracle
from paper_1901_07454_amd import mechgen
from tests import models
from workloads import gen

STEEP = """mechanism steep
parameter g = 1.0
parameter s = 0.1
parameter big = 1.0
state a
state b
rate x = (v + 40) / s
gate a inf 1 / (1 + exp(x)) tau 1 + 1 / (1 + exp(x))
gate b alpha exprelr(x) beta exp(-x / 1000) + 1
current g * a * b * (v / 0.001) * big
"""


def _eval(e, env):
    """A parsed expression in IEEE doubles, overflow and all."""
    k = e[0]
    if k in ("num", "var"):
        return np.float64(e[1] if k == "num" else env[e[1]])
    if k == "neg":
        return -_eval(e[1], env)
    if k == "call":
        x = _eval(e[2], env)
        if e[1] == "exprelr":
            return np.float64(1.0) if 1.0 + x == 1.0 else x / np.expm1(x)
        return getattr(np, e[1])(x)
    a, b = _eval(e[2], env), _eval(e[3], env)
    return {"+": np.add, "-": np.subtract, "*": np.multiply, "/": np.divide}[e[1]](a, b)


def test_device_functions_saturate_as_described(tmp_path):
    """The emitted device functions, compiled for the host (their qualifiers
    defined away), against the description evaluated in IEEE arithmetic: the
    same infinities and no NaN of their own, arguments on both sides of every
    threshold of the exponential.  A few ulp apart otherwise (two math
    libraries, at most ten operations)."""
    m = mechgen.parse_mechanism(STEEP)
    (tmp_path / "hip").mkdir()
    (tmp_path / "gen").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(
        "#pragma once\n#include <cmath>\nusing std::exp; using std::expm1; using std::fma; using std::ldexp;\n"
        "using std::rint;\n#define __device__\n#define __host__\n#define __forceinline__ inline\n")
    (tmp_path / "gen" / "mechanisms_desc.hpp").write_text(mechgen.render_desc([m]))
    (tmp_path / "gen" / "mechanisms.hpp").write_text(mechgen.render_device([m]))
    (tmp_path / "probe.cpp").write_text("""
#include <cstdio>
#include "gen/mechanisms.hpp"
using namespace arbmi::gen;
int main() {
    double v, s, big;
    while (std::scanf("%la %la %la", &v, &s, &big) == 3) {
        double p[2][kMaxParams] = {{1.0, s, big}, {1.0, s, big}}, st[2][kMaxStates] = {{0.3, 0.4}, {0.3, 0.4}};
        double vv[2] = {v, v}, cur[2], one[kMaxStates] = {0.3, 0.4}, c1, c0[2];
        current_pair(0, vv, p, st, c0);
        advance_pair(0, vv, 0.025, p, st, cur);
        advance_one(0, v, 0.025, p[0], one, &c1);
        std::printf("%a %a %a %a %a %a %a\\n", c0[0], st[0][0], st[1][1], cur[1], one[0], one[1], c1);
    }
}
""")
    exe = tmp_path / "probe"
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", f"-I{tmp_path}", str(tmp_path / "probe.cpp"),
                    f"-I{mechgen.OUT_DIR}", "-o", str(exe)], check=True, capture_output=True)
    # (v + 40) / s through the thresholds of exp and expm1, and far past them
    xs = [-1e300, -1e4, -760.0, -745.2, -710.0, -700.0, -1e-20, 0.0, 1.0, 700.0, 708.9, 709.5, 709.7, 709.9, 710.3,
          715.0, 720.0, 800.0, 1e4, 1e300, np.inf, -np.inf]
    rows = [(-40.0 + x if abs(x) > 1e5 else -40.0 + 0.1 * x, 1.0 if abs(x) > 1e5 else 0.1, 1.0) for x in xs]
    rows += [(1e306, 0.1, 1.0), (-1e306, 0.1, 1.0), (30.0, 1e-3, 1e300)]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(float(t).hex() for t in r) for r in rows),
                         capture_output=True, text=True, check=True).stdout.split("\n")
    gate = {g.state: g for g in m.gates}
    dt = 0.025
    with np.errstate(all="ignore"):
        for (v, s, big), line in zip(rows, out):
            got = [float.fromhex(t) for t in line.split()]
            env = {"v": np.float64(v), "g": np.float64(1.0), "s": np.float64(s), "big": np.float64(big)}
            for r, e in m.rates:
                env[r] = _eval(e, env)
            c0 = _eval(m.current, {**env, "a": 0.3, "b": 0.4})
            inf, tau = _eval(gate["a"].a, env), _eval(gate["a"].b, env)
            a = inf + (0.3 - inf) * np.exp(-dt / tau)
            al, be = _eval(gate["b"].a, env), _eval(gate["b"].b, env)
            x = al / (al + be)
            b = x + (0.4 - x) * np.exp(-dt * (al + be))
            cur = _eval(m.current, {**env, "a": a, "b": b})
            np.testing.assert_allclose(got, [c0, a, b, cur, a, b, cur], rtol=1e-13, err_msg=str((v, s)))


@pytest.mark.gpu
@pytest.mark.parametrize("vhalf", [-5000.0, -4390.0, 4000.0])
def test_gate_switched_off_by_its_midpoint(vhalf):
    """hcn with a midpoint thousands of mV away: e^((v - vhalf) / 6) overflows
    (or vanishes) and the gate closes (opens); voltages as the oracle's to the
    suite's 1e-8 mV."""
    from paper_1901_07454_amd import arbmi
    d = models.bare_cell([-1, 0], [8, 5], [150.0, 90.0], [2.0, 1.0])
    d.syn.append((-1, 0, 2.0, 0.0))
    d.ext.append((0, 5, 0.05))
    dens = [(0, b, "hcn", {"gbar": 3e-4, "vhalf": vhalf}) for b in (-1, 0, 1)]
    m = gen.with_densities(gen.assemble([d], n_steps=200), dens)
    ref = oracle.Sim(m)
    ref.run(200)
    sim = arbmi.Simulation(m)
    sim.step(200)
    V = sim.voltages_host()
    sim.close()
    assert np.max(np.abs(V - ref.state()["V"])) <= 1e-8
