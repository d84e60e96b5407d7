"""The forward pass in tile passes (energy and gradient entry points): the
final state of qng_energy_dev, its sign included, against the oracle's forward
pass, at register sizes around the tile edges (12 tile qubits in either
precision; below that the register is one tile, below 10 some threads idle) and
for every gate kind.

Tolerances: every gate rounds an amplitude by a few units u, and M such
roundings add like a random walk, so max|psi - psi_oracle| is held to
8 sqrt(M) u times the largest amplitude (u = 2^-53 or 2^-24), with the same
bound on the gradient's largest entry times the number of terms' norm."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

U = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2011_02991_amd as q
    c = q.Context(0)
    c.set_stream(None)
    yield q, c, torch
    c.close()


def problem(kind, n, seed):
    if kind == "plain":
        return W.random_circuit(n, 40 + 3 * n, seed, n_terms=4)
    if kind == "controlled":
        return W.controlled_circuit(n, 40 + 3 * n, seed, n_terms=4)
    if kind == "strings":
        return W.string_circuit(n, 40, seed, n_terms=4)
    return W.make_problem("layers", n, 3, (W.RY, W.RZ), "cnot_chain", 4, seed)


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("kind,n", [("plain", 1), ("plain", 2), ("plain", 3), ("layers", 9), ("plain", 10),
                                    ("layers", 11), ("plain", 12), ("controlled", 12), ("layers", 13),
                                    ("controlled", 14), ("strings", 13), ("strings", 6), ("plain", 16)])
def test_final_state_and_gradient(env, kind, n, prec):
    q, ctx, torch = env
    for seed in (8101, 8102):
        pr = problem(kind, n, seed + n)
        pr.in_state = W.random_state(n, seed + 50)
        circ = q.Circuit.from_problem(pr)
        ins = torch.tensor(pr.in_state, device="cuda")
        E = torch.zeros((), dtype=torch.float64, device="cuda")
        psi = torch.zeros(2 ** n, dtype=torch.complex128, device="cuda")
        grad = torch.zeros(pr.n_params, dtype=torch.float64, device="cuda")
        ctx.energy_dev(circ, pr.theta, E.data_ptr(), psi.data_ptr(), in_state_dev_ptr=ins.data_ptr(), prec=prec)
        torch.cuda.synchronize()
        want = oracle.forward(pr)
        tol = 8.0 * np.sqrt(max(4, 4 * pr.n_gates)) * U[prec]
        err = np.abs(psi.cpu().numpy() - want).max() / np.abs(want).max()
        print(kind, n, prec, seed, "psi", err, "tol", tol, flush=True)
        assert err <= tol
        e0, g0 = oracle.energy_grad(pr)
        scale = np.abs(pr.coeff).sum()
        assert abs(float(E) - e0) <= tol * scale
        ctx.energy_grad_dev(circ, pr.theta, E.data_ptr(), grad.data_ptr(), in_state_dev_ptr=ins.data_ptr(), prec=prec)
        torch.cuda.synchronize()
        assert abs(float(E) - e0) <= tol * scale
        assert np.abs(grad.cpu().numpy() - g0).max(initial=0.0) <= tol * scale
