"""Registers whose forward state and column starts run with the state in LDS
(up to 13 qubits in complex128, 14 in complex64; the next size takes the launches
per column): metric and gradient against the oracle over one-amplitude-pair
registers, circuits of fewer and more gates than one chunk of steps (64), plain,
controlled and string rotations, all columns in one group and one column per group.

Tolerances (G against its largest entry, the gradient against the terms' norm):
complex128 1e-10; complex64 16 sqrt(4 M) 2^-24 for M gates."""
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


def problem(kind, n, gates, seed):
    if kind == "controlled":
        return W.controlled_circuit(n, gates, seed, n_terms=4)
    if kind == "strings":
        return W.string_circuit(n, gates, seed, n_terms=4)
    return W.random_circuit(n, gates, seed, n_terms=4)


@pytest.mark.parametrize("streams", [0, 1])
@pytest.mark.parametrize("kind,n,gates,prec", [
    ("plain", 1, 5, "c128"), ("plain", 2, 63, "c128"), ("plain", 3, 66, "c64"), ("controlled", 2, 30, "c128"),
    ("controlled", 6, 130, "c128"), ("strings", 5, 30, "c128"), ("plain", 9, 64, "c64"), ("plain", 13, 70, "c128"),
    ("plain", 14, 60, "c128"), ("plain", 14, 60, "c64"), ("controlled", 13, 60, "c64")])
def test_chain(env, kind, n, gates, prec, streams):
    q, ctx = env
    pr = problem(kind, n, gates, 9400 + 7 * n + gates)
    pr.in_state = W.random_state(n, 91)
    want = oracle.step(pr)
    ctx.set_option(q.OPT_COLUMN_STREAMS, streams)
    try:
        res = ctx.step(q.Circuit.from_problem(pr), pr.theta, pr.dt, pr.tikhonov, in_state=pr.in_state, prec=prec)
    finally:
        ctx.set_option(q.OPT_COLUMN_STREAMS, 0)
    tol = 1e-10 if prec == "c128" else 16.0 * np.sqrt(4 * pr.n_gates) * 2.0 ** -24
    for key, scale in (("G", np.abs(want["G"]).max()), ("grad", np.abs(pr.coeff).sum())):
        err = np.abs(res[key] - want[key]).max() / scale
        print(kind, n, gates, prec, streams, key, err, "tol", tol, flush=True)
        assert err <= tol


@pytest.mark.parametrize("tiles", [1, 0])
def test_chain_batched(env, tiles):
    """Members below, at and above the chain's largest register, in one batch;
    one launch per column block (tiles 1) and as many as fit."""
    q, ctx = env
    prs = [problem(kind, n, gates, 9500 + n + gates) for kind, n, gates in
           (("plain", 1, 4), ("controlled", 5, 70), ("plain", 8, 66), ("strings", 9, 20), ("plain", 13, 40),
            ("controlled", 13, 40), ("plain", 14, 40))]
    ctx.set_option(q.OPT_BATCH_TILES, tiles)
    try:
        res = ctx.step_batched([q.Circuit.from_problem(p) for p in prs], [p.theta for p in prs], 0.1, 1e-4)
    finally:
        ctx.set_option(q.OPT_BATCH_TILES, 0)
    for p, r in zip(prs, res):
        want = oracle.step(p)
        for key, scale in (("G", np.abs(want["G"]).max()), ("grad", np.abs(p.coeff).sum())):
            err = np.abs(r[key] - want[key]).max() / scale
            print(p.name, tiles, key, err, flush=True)
            assert err <= 1e-10
