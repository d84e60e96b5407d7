"""Which registers of the chain's sizes take it: few gates between the rotations
on any, many fixed ones on the smallest only (the launches per column with the
forward plan are cheaper there on larger ones), controlled rotations always.
Told by the launches besides the sweeps', and against the oracle on both sides.

Tolerances as for any metric: complex128 1e-10; complex64 16 sqrt(4 M) 2^-24."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

P = 40


@pytest.mark.parametrize("n,prec,fixed,controlled,chain", [
    (6, "c128", 0, False, True), (6, "c128", 10, False, True), (9, "c64", 10, False, True),
    (13, "c128", 0, False, True), (13, "c128", 12, False, False), (14, "c64", 12, False, False),
    (12, "c64", 40, False, False), (13, "c128", 12, True, True), (14, "c64", 12, True, True)])
def test_route(n, prec, fixed, controlled, chain):
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    rng = np.random.default_rng(9900 + n + fixed)
    rows = []
    for p in range(P):
        a, b = (int(x) for x in rng.choice(n, 2, replace=False))
        rows.append((W.CRY, a, b, p) if controlled and p % 4 == 0 else (int(rng.integers(0, 3)), a, -1, p))
        for _ in range(fixed):
            a, b = (int(x) for x in rng.choice(n, 2, replace=False))
            rows.append((W.CZ, a, b, -1))
    pr = W.Problem("fixed%d" % fixed, n, np.asarray(rows, np.int32), rng.uniform(0, 2 * np.pi, P),
                   np.zeros((1, n), np.uint8), np.ones(1))
    pr.in_state = W.random_state(n, 94)
    ctx = q.Context(0)
    G, T = ctx.metric(q.Circuit.from_problem(pr), pr.theta, in_state=pr.in_state, prec=prec)
    stats = ctx.stats()
    ctx.close()
    extra = stats["other_launches"] - stats["sweep_launches"]
    want = oracle.metric(pr)
    tol = 1e-10 if prec == "c128" else 16.0 * np.sqrt(4 * pr.n_gates) * 2.0 ** -24
    err = np.abs(G - want[0]).max() / np.abs(want[0]).max()
    print(n, prec, fixed, controlled, "launches besides the sweeps'", extra, "err", err, "tol", tol, flush=True)
    assert err <= tol
    # a chain is two launches a group of columns; else one or more a column block
    assert extra < 10 if chain else extra >= P // 4


def test_two_threads_of_different_registers():
    """Chains of 13 and 12 qubits (128 and 64 KB of LDS) started by two threads at
    once, each on its own context: bitwise what each gives alone."""
    import threading
    import torch  # noqa: F401
    import paper_2011_02991_amd as q
    prs = [W.make_problem("layers", n, 2, (W.RY, W.RZ), "cnot_chain", 2, 9990 + n) for n in (13, 12)]
    ctxs = [q.Context(0) for _ in prs]
    circs = [q.Circuit.from_problem(p) for p in prs]
    want = [c.metric(k, p.theta)[0] for c, k, p in zip(ctxs, circs, prs)]
    same = [[], []]

    def work(i):
        for _ in range(40):
            same[i].append(np.array_equal(ctxs[i].metric(circs[i], prs[i].theta)[0], want[i]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for c in ctxs:
        c.close()
    assert [len(s) for s in same] == [40, 40] and all(same[0]) and all(same[1])
