"""The steps' solve on the device: what the statistics, the errors and the
workspace limits of a call say of it."""
import re
import time

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

EPS, DT = 1e-2, 0.1


@pytest.fixture(scope="module")
def env():
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    return q


def problem(P, seed=8400):
    return W.random_circuit(6, P, seed + P, fixed_fraction=0.0, n_terms=5)


def check(r, P):
    """Cholesky's backward error, a modest multiple of P u, amplified by the condition number."""
    A = r["G"].real + EPS * np.eye(P)
    want = np.linalg.solve(A, -DT * r["grad"])
    err, tol = np.linalg.norm(r["dtheta"] - want), 8 * P * 2.0 ** -53 * np.linalg.cond(A) * np.linalg.norm(want)
    print("P", P, "err", err, "tol", tol, flush=True)
    assert err <= tol


def test_batch_statistics(env):
    """The solve's time is in solve_ms: at 300 parameters it is 20 launches, each
    waiting for the one before, which no device does in 0.05 ms (without G outputs
    nothing else that the call does after them takes as long)."""
    q = env
    ctx = q.Context(0)
    prs = [problem(300, 8400 + k) for k in range(3)]
    circs = [q.Circuit.from_problem(p) for p in prs]
    for _ in range(2):
        t0 = time.perf_counter()
        res = ctx.step_batched(circs, [p.theta for p in prs], DT, EPS, want_G=False)
        wall = 1e3 * (time.perf_counter() - t0)
    s = ctx.stats()
    ctx.close()
    print(s, wall, flush=True)
    assert s["solve_ms"] >= 0.05
    assert s["metric_ms"] + s["grad_ms"] + s["solve_ms"] <= wall
    assert all(r["G"] is None and np.isfinite(r["dtheta"]).all() for r in res)


@pytest.mark.parametrize("zero", [3, 31, 32, 97, 143])
def test_bad_pivot_is_named(env, zero):
    """A rotation controlled by a qubit left in |0>, an exactly zero row of G: the
    device solve's error names the pivot that the host's solve of the same G does,
    alone and in a batch."""
    q = env
    ctx = q.Context(0)
    pr = W.make_problem("layers", 9, 8, (W.RX, W.RY), "cz_ring", 4, 8450)
    gates = np.insert(pr.gates, 0, [W.CRX, 9, 0, zero], axis=0)
    gates[1:, 3] += gates[1:, 3] >= zero
    P = pr.n_params + 1
    circ = q.Circuit(10, gates, P, np.pad(pr.pauli, ((0, 0), (0, 1))), pr.coeff)
    theta = np.insert(pr.theta, zero, 0.3)
    G, _ = ctx.metric(circ, theta)
    with pytest.raises(q.QNGError) as host:
        q.solve_shifted(G, 0.0, np.ones(P))
    assert host.value.name == "QNG_E_NOT_SPD" and "pivot %d)" % zero in str(host.value)
    with pytest.raises(q.QNGError) as e:
        ctx.step(circ, theta, DT, 0.0)
    print(zero, e.value, flush=True)
    assert str(e.value) == str(host.value)
    good = q.Circuit.from_problem(pr)
    with pytest.raises(q.QNGError) as e:
        ctx.step_batched([good, circ], [pr.theta, theta], DT, 0.0)
    assert e.value.name == "QNG_E_NOT_SPD" and "ansatz 1: " in str(e.value) and "pivot %d)" % zero in str(e.value)
    ctx.close()


def least_workspace(q, ctx, call):
    """Bytes of the call's workspace with every part that it can do without left out
    (one column block at a time: how many go together depends on the limit)."""
    ctx.set_option(q.OPT_COLUMN_STREAMS, 1)
    ctx.set_mem_limit(1)
    with pytest.raises(q.QNGError) as e:
        call()
    assert e.value.name == "QNG_E_OUT_OF_MEMORY"
    return int(re.search(r"workspace of (\d+) bytes", str(e.value)).group(1))


def test_step_without_room_for_the_solve(env):
    """A limit with no room for the device solve's matrix nor for the images of the
    forward pass behind the metric (9 gates): the host solve of the same G.  The
    device step, which has to solve on the device, does not fit."""
    q = env
    import torch
    ctx = q.Context(0)
    pr = W.make_problem("layers", 9, 8, (W.RX, W.RY), "cz_ring", 4, 8460)
    P = pr.n_params
    assert P ** 3 >= 128 ** 3
    circ = q.Circuit.from_problem(pr)
    want = ctx.step(circ, pr.theta, DT, EPS)
    check(want, P)
    ctx.set_mem_limit(least_workspace(q, ctx, lambda: ctx.step(circ, pr.theta, DT, EPS)))
    got = ctx.step(circ, pr.theta, DT, EPS)
    x = torch.zeros(P, dtype=torch.float64, device="cuda")
    with pytest.raises(q.QNGError) as e:
        ctx.step_dev(circ, pr.theta, DT, EPS, x.data_ptr())
    assert e.value.name == "QNG_E_OUT_OF_MEMORY"
    ctx.close()
    check(got, P)
    assert np.abs(got["G"] - want["G"]).max() <= 1e-12 and np.abs(got["grad"] - want["grad"]).max() <= 1e-12


def test_batch_without_room_for_the_solves(env):
    q = env
    ctx = q.Context(0)
    prs = [problem(P, 8470) for P in (40, 130, 7)]
    circs, thetas = [q.Circuit.from_problem(p) for p in prs], [p.theta for p in prs]
    want = ctx.step_batched(circs, thetas, DT, EPS)
    ctx.set_mem_limit(least_workspace(q, ctx, lambda: ctx.step_batched(circs, thetas, DT, EPS)))
    got = ctx.step_batched(circs, thetas, DT, EPS)
    ctx.close()
    for p, g, w in zip(prs, got, want):
        check(g, p.n_params)
        check(w, p.n_params)
        assert np.abs(g["G"] - w["G"]).max() <= 1e-12 and g["E"] == w["E"]


@pytest.mark.parametrize("strings", [False, True])
def test_energy_without_room_for_the_plan(env, strings):
    """A limit with room for the registers alone: the energy runs gate by gate (a
    string is one kernel then); without one, in fewer launches."""
    q = env
    import torch
    import oracle
    ctx = q.Context(0)
    pr = W.string_layers(8, 2, 4, 8480) if strings else W.make_problem("layers", 9, 8, (W.RX, W.RY), "cz_ring", 4, 8481)
    circ = q.Circuit.from_problem(pr)
    E = torch.zeros((), dtype=torch.float64, device="cuda")
    psi = torch.zeros(2 ** pr.n_qubits, dtype=torch.complex128, device="cuda")
    call = lambda: ctx.energy_dev(circ, pr.theta, E.data_ptr(), psi.data_ptr())
    tol = 8.0 * np.sqrt(4 * pr.n_gates) * 2.0 ** -53
    for limited in (False, True):
        if limited:
            ctx.set_mem_limit(least_workspace(q, ctx, call))
        call()
        torch.cuda.synchronize()
        launches = ctx.stats()["other_launches"]
        print(strings, limited, "gates", pr.n_gates, "launches", launches, flush=True)
        want = oracle.forward(pr)
        assert np.abs(psi.cpu().numpy() - want).max() <= tol * np.abs(want).max()
        assert abs(float(E) - oracle.energy(pr)) <= tol * np.abs(pr.coeff).sum()
        assert launches == pr.n_gates + 4 if limited else launches < pr.n_gates
    ctx.close()


def test_optional_solve_takes_no_kept_state(env):
    """The derivative-state variant at a limit with room for all its states but not
    for the solve's matrix as well: all are kept, and the host solves."""
    q = env
    ctx = q.Context(0)
    ctx.set_option(q.OPT_METHOD, 1)
    pr = W.make_problem("layers", 9, 8, (W.RX, W.RY), "cz_ring", 4, 8490)
    P = pr.n_params
    circ = q.Circuit.from_problem(pr)
    call = lambda: ctx.step(circ, pr.theta, DT, EPS)
    ctx.set_option(q.OPT_STATE_CHUNK, P)
    limit = least_workspace(q, ctx, call)
    ctx.set_option(q.OPT_STATE_CHUNK, 0)
    ctx.set_mem_limit(limit)
    got = call()
    chunks = ctx.stats()["state_chunks"]
    ctx.close()
    print(limit, chunks, flush=True)
    assert chunks == 1
    check(got, P)
