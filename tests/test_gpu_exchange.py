"""The sweep's exchanges between thread mappings, at tile sizes whose tiles take
part of a wavefront, one, two and four of them (the wavefront bits of a mapping
stand still over most exchanges, which then need no barrier): random circuits
over tiles of 6 to 12 qubits against the oracle's metric and gradient.

Tolerances: complex128 1e-10; complex64 16 sqrt(4 M) 2^-24 for M gates."""
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


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("tile,block", [(6, 1), (8, 1), (9, 1), (10, 1), (10, 2), (11, 1), (11, 2), (11, 4), (12, 1),
                                        (12, 2)])
def test_exchanges(env, tile, block, prec):
    q, ctx = env
    pr = W.random_circuit(13, 90, 9300 + 17 * tile + block, n_terms=4)
    want = oracle.step(pr)
    ctx.set_option(q.OPT_TILE_QUBITS, tile)
    ctx.set_option(q.OPT_BLOCK_COLUMNS, block)
    try:
        res = ctx.step(q.Circuit.from_problem(pr), pr.theta, pr.dt, pr.tikhonov, prec=prec)
    finally:
        ctx.set_option(q.OPT_TILE_QUBITS, 0)
        ctx.set_option(q.OPT_BLOCK_COLUMNS, 0)
    tol = 1e-10 if prec == "c128" else 16.0 * np.sqrt(4 * pr.n_gates) * 2.0 ** -24
    for key, scale in (("G", np.abs(want["G"]).max()), ("grad", np.abs(pr.coeff).sum())):
        err = np.abs(res[key] - want[key]).max() / scale
        print(tile, block, prec, key, err, "tol", tol, flush=True)
        assert err <= tol


@pytest.mark.parametrize("n", [15, 16, 17])
def test_tile_sums(env, n):
    """Sums over 128, 256 and 512 tiles (one wavefront up to 256, then 1024
    threads)."""
    q, ctx = env
    pr = W.random_circuit(n, 14, 9350 + n, n_terms=3)
    want = oracle.step(pr)
    ctx.set_option(q.OPT_TILE_QUBITS, 8)
    try:
        res = ctx.step(q.Circuit.from_problem(pr), pr.theta, pr.dt, pr.tikhonov)
    finally:
        ctx.set_option(q.OPT_TILE_QUBITS, 0)
    for key, scale in (("G", np.abs(want["G"]).max()), ("grad", np.abs(pr.coeff).sum())):
        err = np.abs(res[key] - want[key]).max() / scale
        print(n, key, err, flush=True)
        assert err <= 1e-10
