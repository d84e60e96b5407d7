"""Layers of CZ gates on every pair of qubits, which the sweep runs as sets (one
sign per amplitude from up to 24 CZs): registers of one tile and of several
(12 tile qubits), layers of 1, 3, 24, 25 and more CZs, CZs on register, thread
and base bits of the tile, repeated pairs (which cancel), every block width, both
precisions, against the oracle's metric and gradient.

Tolerances (G against its largest entry, the gradient against the terms' norm):
complex128 1e-10; complex64 16 sqrt(4 M) 2^-24 for M
gates (each rounds an amplitude a few times, like a random walk; two states in a
product)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    c = q.Context(0)
    yield q, c
    c.close()


def layers(n, czs, n_layers, seed):
    rng = np.random.default_rng(seed)
    rows, p = [], 0
    for _ in range(n_layers):
        for qubit in rng.permutation(n)[:4]:
            rows.append([int(rng.integers(W.RX, W.RZ + 1)), int(qubit), -1, p])
            p += 1
        for _ in range(czs):
            a, b = rng.choice(n, size=2, replace=False)
            rows.append([W.CZ, int(a), int(b), -1])
    theta, pauli, coeff = W.draw_problem_data(seed, p, n, 4)
    return W.Problem(name=f"czs_n{n}_{czs}", n_qubits=n, gates=np.asarray(rows, dtype=np.int32).reshape(-1, 4),
                     theta=theta, pauli=pauli, coeff=coeff, seed=seed)


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("block", [1, 2, 4])
@pytest.mark.parametrize("n,czs", [(2, 3), (5, 10), (10, 24), (12, 25), (13, 1), (13, 49), (14, 30)])
def test_cz_layers(env, n, czs, block, prec):
    q, ctx = env
    pr = layers(n, czs, 4, 9200 + 31 * n + czs)
    pr.in_state = W.random_state(n, 77)
    want = oracle.step(pr)
    ctx.set_option(q.OPT_BLOCK_COLUMNS, block)
    try:
        res = ctx.step(q.Circuit.from_problem(pr), pr.theta, pr.dt, pr.tikhonov, in_state=pr.in_state, prec=prec)
    finally:
        ctx.set_option(q.OPT_BLOCK_COLUMNS, 0)
    tol = 1e-10 if prec == "c128" else 16.0 * np.sqrt(4 * pr.n_gates) * 2.0 ** -24
    for key, scale in (("G", np.abs(want["G"]).max()), ("grad", np.abs(pr.coeff).sum())):
        err = np.abs(res[key] - want[key]).max() / scale
        print(n, czs, block, prec, key, err, "tol", tol, flush=True)
        assert err <= tol
