"""A batch's members have the same metric, T-dependent gradient and energy bits
whatever ansaetze share their launches: alone, and beside members whose registers
have more tiles (256 against 512 among them; complex64 and complex128; G outputs, so nothing is solved
from the compared values)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_bits_do_not_depend_on_the_company(prec):
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    small = [W.make_problem("small", n, 2, (W.RY, W.RZ), "cnot_chain", 4, 9950 + n) for n in (12, 15, 19)]
    big = W.make_problem("big", 20, 1, (W.RX, W.RY), "cz_ring", 4, 9960)
    ctx = q.Context(0)

    def run(prs):
        return ctx.step_batched([q.Circuit.from_problem(p) for p in prs], [p.theta for p in prs], 0.1, 1e-2, prec=prec)

    together = run(small + [big])
    for k, pr in enumerate(small):
        alone = run([pr])[0]
        print(prec, pr.n_qubits, np.abs(alone["G"] - together[k]["G"]).max(), flush=True)
        assert np.array_equal(alone["G"], together[k]["G"])
        assert np.array_equal(alone["grad"], together[k]["grad"]) and alone["E"] == together[k]["E"]
    ctx.close()
