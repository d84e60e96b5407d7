"""One context that steps through more distinct circuits than its plan cache
keeps: every result is bitwise that of a context of its own."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_steps_over_distinct_circuits():
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    ctx = q.Context(0)
    for k in range(140):
        # a rotation on each of 4 qubits, then k in binary as CNOTs and CZs (8
        # gates behind the last rotation: three plans a circuit)
        gates = [(W.RY, a, -1, a) for a in range(4)]
        gates += [(W.CZ if (k >> b) & 1 else W.CNOT, b % 4, (b + 1) % 4, -1) for b in range(9)]
        rng = np.random.default_rng(9700 + k)
        circ = q.Circuit(4, gates, 4, rng.integers(0, 4, (3, 4)), rng.standard_normal(3))
        theta = rng.uniform(0, 2 * np.pi, 4)
        got = ctx.step(circ, theta, 0.1, 1e-3)
        if k % 20 == 5 or k in (84, 85, 86, 127, 128, 129):
            other = q.Context(0)
            want = other.step(circ, theta, 0.1, 1e-3)
            other.close()
            print(k, got["E"], flush=True)
            assert got["E"] == want["E"]
            for key in ("dtheta", "G", "grad"):
                assert np.array_equal(got[key], want[key])
    ctx.close()
