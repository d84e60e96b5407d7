"""The device solve of the steps in panels of 32 columns: parameter counts
around the panel edges, alone (host and device step) and in a batch of unequal
sizes, against numpy's solve of the returned G and gradient; and a zero pivot
in a later panel.

Tolerance: Cholesky's backward error is a modest multiple of P u, amplified by
the condition number, so ||x - x_ref|| <= 8 P u kappa ||x_ref|| (u = 2^-53)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

EPS, DT = 1e-2, 0.1


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2011_02991_amd as q
    c = q.Context(0)
    yield q, c, torch
    c.close()


def problem(P, seed=8200):
    return W.random_circuit(6, P, seed + P, fixed_fraction=0.0, n_terms=5)


def check(r, P):
    A = r["G"].real + EPS * np.eye(P)
    want = np.linalg.solve(A, -DT * r["grad"])
    err = np.linalg.norm(r["dtheta"] - want)
    tol = 8 * P * 2.0 ** -53 * np.linalg.cond(A) * np.linalg.norm(want)
    print("P", P, "err", err, "tol", tol, flush=True)
    assert err <= tol


SIZES = [1, 2, 31, 32, 33, 63, 64, 65, 97, 130]


@pytest.mark.parametrize("P", SIZES)
def test_panel_edges(env, P):
    q, ctx, torch = env
    pr = problem(P)
    circ = q.Circuit.from_problem(pr)
    r = ctx.step(circ, pr.theta, DT, EPS)
    check(r, P)
    no_G = ctx.step(circ, pr.theta, DT, EPS, want_G=False)
    assert no_G["G"] is None and np.abs(no_G["dtheta"] - r["dtheta"]).max() <= 1e-10 * np.abs(r["dtheta"]).max()
    out = [torch.zeros(P, dtype=torch.float64, device="cuda"), torch.zeros(P, P, dtype=torch.complex128, device="cuda"),
           torch.zeros(P, dtype=torch.float64, device="cuda")]
    torch.cuda.synchronize()
    ctx.step_dev(circ, pr.theta, DT, EPS, *[o.data_ptr() for o in out])
    ctx.synchronize()
    check({"dtheta": out[0].cpu().numpy(), "G": out[1].cpu().numpy(), "grad": out[2].cpu().numpy()}, P)


def test_batch_of_unequal_sizes(env):
    q, ctx, _ = env
    prs = [problem(P, 8300) for P in SIZES]
    res = ctx.step_batched([q.Circuit.from_problem(p) for p in prs], [p.theta for p in prs], DT, EPS)
    for r, P in zip(res, SIZES):
        check(r, P)


def test_limit_without_room_for_the_solve(env):
    """A workspace limit that the step met before it solved on the device."""
    q, _, _ = env
    ctx = q.Context(0)
    pr = problem(65)
    circ = q.Circuit.from_problem(pr)
    want = ctx.step(circ, pr.theta, DT, EPS)
    lo, hi = 1 << 10, 1 << 26
    while hi - lo > 256:          # the smallest limit under which the step runs
        mid = (lo + hi) // 2
        ctx.set_mem_limit(mid)
        try:
            ctx.step(circ, pr.theta, DT, EPS)
            hi = mid
        except q.QNGError as e:
            assert e.name == "QNG_E_OUT_OF_MEMORY"
            lo = mid
    ctx.set_mem_limit(hi)
    got = ctx.step(circ, pr.theta, DT, EPS)
    ctx.close()
    check(got, 65)
    assert np.abs(got["G"] - want["G"]).max() <= 1e-12


@pytest.mark.parametrize("zero", [5, 40, 69])
def test_zero_pivot_in_a_later_panel(env, zero):
    """An RZ on a qubit left in |0>: a zero row of G at any place."""
    q, ctx, torch = env
    pr = problem(69)
    gates = pr.gates.copy()
    gates[:, 3] += gates[:, 3] >= zero
    gates = np.insert(gates, zero, [W.RZ, 6, -1, zero], axis=0)
    bad = W.Problem("zero", 7, gates, np.insert(pr.theta, zero, 0.3), np.pad(pr.pauli, ((0, 0), (0, 1))), pr.coeff)
    circ = q.Circuit.from_problem(bad)
    with pytest.raises(q.QNGError) as e:
        ctx.step(circ, bad.theta, DT, 0.0)
    assert e.value.name == "QNG_E_NOT_SPD"
    x = torch.zeros(70, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with pytest.raises(q.QNGError) as e:
        ctx.step_dev(circ, bad.theta, DT, 0.0, x.data_ptr())
    assert e.value.name == "QNG_E_NOT_SPD" and not x.any()
    good = problem(130)      # (large enough for the batch to be solved on the device)
    with pytest.raises(q.QNGError) as e:
        ctx.step_batched([q.Circuit.from_problem(good), circ], [good.theta, bad.theta], DT, 0.0)
    assert e.value.name == "QNG_E_NOT_SPD"
    check(ctx.step(circ, bad.theta, DT, EPS), 70)
