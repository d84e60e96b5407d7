"""Performance cases of the quantum-natural-gradient library: what a program
that optimises an ansatz calls, from the smallest registers (where launches and
latency count) to the largest (where arithmetic and memory traffic do).

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges,
``prepare(case, seed)`` builds what the program holds before a call (the
circuit with its Hamiltonian, the angles, a library context, output buffers),
``run(state)`` is one call, ``exact(case, seed)`` the same results from plain
torch in 64 bits, ``work(case)`` the bytes and operations of one call.

A case is
  op      step      Context.step: host results, one natural-gradient step
          step_dev  Context.step_dev: device results, asynchronous
          metric    Context.metric_dev: G and T
          grad      Context.energy_grad_dev: E and its gradient
          autograd  torch_energy.energy, forward and backward
          batch     Context.step_batched: `members` ansaetze of n .. n_hi qubits
          states    step_dev with the derivative-state method
  ansatz  ry_rz_cnot, rx_ry_cz, rx_ry_rz_cz (layers of rotations on every
          qubit, then the entangler), controlled (RY layer and a ring of
          controlled rotations), strings (RX layer, ZZ on neighbours, one
          X Y..Y X string), shared (two angles per layer)
  prec    c128 or c64 (storage of the registers).  Results of a c64 call carry
          single precision, and the program keeps them as such.
  want_G  a step that returns G as well (then the complex G is formed)
  in_state  the register starts from a given normalised state instead of |0..0>
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2011_02991_amd as qng
from paper_2011_02991_amd import torch_energy

RX, RY, RZ, CNOT, CZ, CRX, CRY, CRZ, RPAULI = range(9)

# The ranges' ends: elements x amplitudes of the largest listed step.
LARGEST = 432 * 431 / 2 * 2.0 ** 24


def listed():
    return [
        # the smallest whole step: 10 qubits, 80 parameters, everything on the host
        dict(name="step_n10_c128", op="step", ansatz="ry_rz_cnot", n=10, layers=4, terms=20, prec="c128", want_G=True),
        # one iteration of a plain variational loop on a small register
        dict(name="grad_n12_c128", op="grad", ansatz="rx_ry_cz", n=12, layers=6, terms=30, prec="c128"),
        # a metric alone (geometry, imaginary time), odd register, complex G
        dict(name="metric_n17_c64", op="metric", ansatz="rx_ry_rz_cz", n=17, layers=5, terms=1, prec="c64"),
        # Pauli-string (ZZ and ladder) ansatz
        dict(name="step_strings_n19_c128", op="step_dev", ansatz="strings", n=19, layers=3, terms=30, prec="c128"),
        # differentiable energy inside a torch program
        dict(name="autograd_n20_c128", op="autograd", ansatz="rx_ry_cz", n=20, layers=10, terms=50, prec="c128"),
        # the ordinary step: 20 qubits, 400 parameters
        dict(name="step_n20_c128", op="step", ansatz="rx_ry_cz", n=20, layers=10, terms=50, prec="c128"),
        # controlled rotations in single precision, odd register
        dict(name="step_controlled_n21_c64", op="step_dev", ansatz="controlled", n=21, layers=4, terms=30, prec="c64"),
        # the step that also returns the complex G, double precision
        dict(name="step_n22_c128_G", op="step_dev", ansatz="ry_rz_cnot", n=22, layers=6, terms=50, prec="c128", want_G=True),
        # derivative states kept (the method that trades memory for time)
        dict(name="states_n22_c64", op="states", ansatz="ry_rz_cnot", n=22, layers=8, terms=50, prec="c64"),
        # many small ansaetze at once
        dict(name="batch48_n8_16_c128", op="batch", ansatz="ry_rz_cnot", n=8, n_hi=16, members=48, layers=4, terms=12, prec="c128"),
        # gradient of a large register from a given state, single precision
        dict(name="grad_n25_c64", op="grad", ansatz="ry_rz_cnot", n=25, layers=8, terms=100, prec="c64", in_state=True),
        # the largest: 24 qubits, 432 parameters, single precision
        dict(name="step_n24_c64", op="step_dev", ansatz="rx_ry_rz_cz", n=24, layers=6, terms=80, prec="c64"),
    ]


def draw(rng):
    while True:
        op = rng.choice(["step", "step", "step_dev", "step_dev", "metric", "grad", "grad", "autograd", "batch", "states"])
        prec = rng.choice(["c128", "c64"])
        ansatz = rng.choice(["ry_rz_cnot", "rx_ry_cz", "rx_ry_rz_cz", "ry_rz_cnot", "rx_ry_cz", "rx_ry_rz_cz",
                             "controlled", "strings", "shared"])
        c = dict(op=op, ansatz=ansatz, prec=prec)
        if op == "batch":
            c["ansatz"] = rng.choice(["ry_rz_cnot", "rx_ry_cz"])
            c["n"] = rng.randint(8, 14)
            c["n_hi"] = c["n"] + rng.randint(0, 6)
            c["members"] = rng.randint(8, 64)
            c["layers"] = rng.randint(2, 6)
        elif op in ("grad", "autograd"):
            c["n"] = rng.randint(6, 25 if prec == "c64" else 24)
            c["layers"] = rng.randint(2, 12)
        elif op == "states":
            c["n"] = rng.randint(12, 22)
            c["layers"] = rng.randint(2, 8)
        else:
            c["n"] = rng.randint(8, 24 if prec == "c64" else 23)
            c["layers"] = rng.randint(2, 10)
        c["terms"] = rng.randint(8, 100)
        if op in ("step", "step_dev"):
            c["want_G"] = rng.random() < 0.3
        if op in ("grad", "step_dev") and rng.random() < 0.25:
            c["in_state"] = True
        if op in ("grad", "autograd"):
            return c
        if _elements_amps(c) * (2 if prec == "c128" else 1) <= 0.6 * LARGEST:
            return c


# ------------------------------------------------------------------ problems

def _gates(ansatz, n, layers):
    """(gates, strings, number of parameters) of a layered ansatz."""
    rows, strings, p = [], [], 0
    if ansatz == "strings":
        for q in range(n - 1):
            s = np.zeros(n, np.uint8)
            s[q] = s[q + 1] = 3
            strings.append(s)
        s = np.full(n, 2, np.uint8)
        s[0] = s[n - 1] = 1
        strings.append(s)
    for layer in range(layers):
        if ansatz == "controlled":
            for q in range(n):
                rows.append((RY, q, -1, p)); p += 1
            for q in range(n - 1):
                rows.append((CRZ, q, q + 1, p)); p += 1
            rows.append((CRX, n - 1, 0, p)); p += 1
        elif ansatz == "strings":
            for q in range(n):
                rows.append((RX, q, -1, p)); p += 1
            for k in range(n):
                rows.append((RPAULI, k, -1, p)); p += 1
        elif ansatz == "shared":
            for j, kind in enumerate((RX, RZ)):
                for q in range(n):
                    rows.append((kind, q, -1, 2 * layer + j))
                if j == 0:
                    rows += [(CNOT, q, q + 1, -1) for q in range(n - 1)]
            p = 2 * layers
        else:
            kinds = {"ry_rz_cnot": (RY, RZ), "rx_ry_cz": (RX, RY), "rx_ry_rz_cz": (RX, RY, RZ)}[ansatz]
            for kind in kinds:
                for q in range(n):
                    rows.append((kind, q, -1, p)); p += 1
            if ansatz == "ry_rz_cnot":
                rows += [(CNOT, q, q + 1, -1) for q in range(n - 1)]
            elif n > 2:
                rows += [(CZ, q, (q + 1) % n, -1) for q in range(n)]
    return np.asarray(rows, np.int32), (np.asarray(strings, np.uint8) if strings else None), p


def _members(case):
    """(n, layers) of every ansatz of the call (one, or a batch's)."""
    if case["op"] != "batch":
        return [(case["n"], case["layers"])]
    r = np.random.default_rng(7300 + case["n"] + 100 * case["n_hi"] + 10000 * case["members"])
    ns = r.integers(case["n"], case["n_hi"] + 1, case["members"])
    ls = r.integers(2, 2 * case["layers"] - 1, case["members"])   # depths around `layers`
    return [(int(a), int(b)) for a, b in zip(ns, ls)]


def _problems(case, seed):
    """The inputs, from the seed alone: angles uniform in [0, 2 pi), Pauli
    letters uniform, coefficients standard normal, states Gaussian.  The first
    term is the constant offset that a physical Hamiltonian carries."""
    out = []
    rng = np.random.default_rng(seed)
    for n, layers in _members(case):
        gates, strings, P = _gates(case["ansatz"], n, layers)
        pr = dict(n=n, gates=gates, strings=strings, P=P, theta=rng.uniform(0.0, 2.0 * math.pi, P),
                  pauli=rng.integers(0, 4, (case["terms"], n)).astype(np.uint8),
                  coeff=rng.standard_normal(case["terms"]), in_state=None)
        pr["pauli"][0], pr["coeff"][0] = 0, 0.25
        if case.get("in_state"):
            dev = "cuda" if torch.cuda.is_available() else "cpu"
            g = torch.Generator(device=dev).manual_seed(seed)
            v = torch.randn(2 ** n, 2, generator=g, device=dev, dtype=torch.float64)
            v /= v.norm()
            v /= v.norm()
            pr["in_state"] = torch.view_as_complex(v)
        out.append(pr)
    return out


def _step_size(case):
    """(dt, tikhonov).  A single-precision metric is solved with a stronger
    shift: the solve amplifies the metric's rounding by 1 / shift."""
    return 0.1, (1e-4 if case["prec"] == "c128" else 1e-1)


def prepare(case, seed):
    prs = _problems(case, seed)
    circs = [qng.Circuit(p["n"], p["gates"], p["P"], p["pauli"], p["coeff"], p["strings"]) for p in prs]
    dt, eps = _step_size(case)
    st = dict(case=case, circs=circs, thetas=[p["theta"] for p in prs], dt=dt, eps=eps, prec=case["prec"])
    op, c, P = case["op"], circs[0], prs[0]["P"]
    # host results come back on the context's own stream; device results stay
    # on the caller's stream
    st["ctx"] = ctx = qng.Context(0)
    if op not in ("step", "batch"):
        ctx.set_stream(torch.cuda.current_stream().cuda_stream or None)
        st["in_state"] = prs[0]["in_state"]
        f64 = dict(dtype=torch.float64, device="cuda")
        st["E"] = torch.zeros((), **f64)
        st["grad"], st["dtheta"] = torch.zeros(P, **f64), torch.zeros(P, **f64)
        if op == "metric" or case.get("want_G"):
            st["G"] = torch.zeros(P, P, dtype=torch.complex128, device="cuda")
        if op == "metric":
            st["T"] = torch.zeros(P, dtype=torch.complex128, device="cuda")
        st["status"] = torch.zeros((), dtype=torch.int32, device="cuda")
        if op == "states":
            ctx.set_option(qng.OPT_METHOD, 1)
        if op == "autograd":
            st["theta_t"] = torch.tensor(prs[0]["theta"], dtype=torch.float64, requires_grad=True)
    return st


_SINGLE = {torch.float64: torch.float32, torch.complex128: torch.complex64,
           np.dtype(np.float64): np.float32, np.dtype(np.complex128): np.complex64}


def _kept(st, out):
    """What the program keeps: results of a c64 call in single precision."""
    if st["prec"] == "c128":
        return out
    conv = {}
    for k, v in out.items():
        if isinstance(v, torch.Tensor) and v.dtype in _SINGLE:
            v = v.to(_SINGLE[v.dtype])
        elif isinstance(v, np.ndarray):
            v = v.astype(_SINGLE[v.dtype])
        conv[k] = v
    return conv


def run(st):
    op, ctx, c, th, prec = st["case"]["op"], st["ctx"], st["circs"][0], st["thetas"][0], st["prec"]
    if op == "step":
        r = ctx.step(c, th, st["dt"], st["eps"], prec=prec, want_G=bool(st["case"].get("want_G")))
        if r["G"] is None:
            del r["G"]
        return _kept(st, r)
    if op == "batch":
        rs = ctx.step_batched(st["circs"], st["thetas"], st["dt"], st["eps"], prec=prec, want_G=False)
        return _kept(st, {"dtheta": np.concatenate([r["dtheta"] for r in rs]),
                          "grad": np.concatenate([r["grad"] for r in rs]),
                          "E": np.asarray([r["E"] for r in rs])})
    if op == "autograd":
        t = st["theta_t"]
        t.grad = None
        E = torch_energy.energy(ctx, c, t, prec=prec)
        E.backward()
        return _kept(st, {"E": E.detach(), "grad": t.grad})
    ins = st["in_state"].data_ptr() if st["in_state"] is not None else None
    if op == "metric":
        ctx.metric_dev(c, th, st["G"].data_ptr(), st["T"].data_ptr(), in_state_dev_ptr=ins, prec=prec)
        return _kept(st, {"G": st["G"], "T": st["T"]})
    if op == "grad":
        ctx.energy_grad_dev(c, th, st["E"].data_ptr(), st["grad"].data_ptr(), in_state_dev_ptr=ins, prec=prec)
        return _kept(st, {"E": st["E"], "grad": st["grad"]})
    # step_dev, states
    ctx.step_dev(c, th, st["dt"], st["eps"], st["dtheta"].data_ptr(), st["G"].data_ptr() if "G" in st else None,
                 st["grad"].data_ptr(), st["E"].data_ptr(), st["status"].data_ptr(), in_state_dev_ptr=ins, prec=prec)
    out = {"dtheta": st["dtheta"], "grad": st["grad"], "E": st["E"], "status": st["status"]}
    if "G" in st:
        out["G"] = st["G"]
    return _kept(st, out)


# ------------------------------------------------------------------ work

def _rotations(case, n, layers):
    per = {"ry_rz_cnot": 2, "rx_ry_cz": 2, "rx_ry_rz_cz": 3, "controlled": 2, "strings": 2, "shared": 2}
    return per[case["ansatz"]] * n * layers


def _elements_amps(case):
    return float(sum(r * (r - 1) / 2 * 2.0 ** n
                     for n, r in ((n, _rotations(case, n, l)) for n, l in _members(case))))


def work(case):
    """Metric: one inner product (4 operations per amplitude for its real part,
    8 complex) per pair of rotations; the states they are taken between, one
    per rotation, each gate applied (6) to those above it once.  Energy and
    gradient: forward, Hamiltonian and reverse sweep.  Bytes: the inputs, the
    results and one register each of psi and H psi."""
    amp = 16 if case["prec"] == "c128" else 8
    byts = flops = 0.0
    for n, layers in _members(case):
        R, V = _rotations(case, n, layers), 2.0 ** n
        P = 2 * layers if case["ansatz"] == "shared" else R
        if case["op"] != "metric":
            flops += V * (6.0 * case["terms"] + R * (6 + 2 * 6 + 8))
            byts += 2 * V * amp + 8 * P
        if case["op"] not in ("grad", "autograd"):
            cplx = case["op"] == "metric" or case.get("want_G")
            flops += V * R * (R - 1) / 2 * ((8 if cplx else 4) + 6)
            byts += V * amp + 8 * P + (16 * P * P if cplx else 0)
        if case.get("in_state"):
            byts += 16 * V
    return {"bytes": byts, "flops": flops}


# ------------------------------------------------------------------ exact

def _bits(S, n, q):
    """S (k, 2^n) as (k, high, 2, low) around qubit q."""
    return S.view(S.shape[0], 2 ** (n - 1 - q), 2, 2 ** q)


def _pauli(S, n, q, letter):
    v = _bits(S, n, q)
    if letter == 3:
        v[:, :, 1] *= -1
        return
    a, b = v[:, :, 0].clone(), v[:, :, 1]
    if letter == 1:
        v[:, :, 0] = b
        v[:, :, 1] = a
    else:
        v[:, :, 0] = -1j * b
        v[:, :, 1] = 1j * a


def _rotate(v, kind, t):
    """exp(i t sigma / 2) on the axis of v (.., .., 2, ..) in place."""
    c, s = math.cos(t / 2), math.sin(t / 2)
    if kind == RZ:
        v[:, :, 0] *= complex(c, s)
        v[:, :, 1] *= complex(c, -s)
        return
    f, g = (1j * s, 1j * s) if kind == RX else (s, -s)
    a, b = v[:, :, 0], v[:, :, 1]
    na = c * a
    na += f * b
    b *= c
    b += g * a
    v[:, :, 0] = na


def _apply(S, n, g, t, strings):
    """Gate g (angle t) on every row of S in place."""
    kind, q0, q1 = int(g[0]), int(g[1]), int(g[2])
    if kind <= RZ:
        _rotate(_bits(S, n, q0), kind, t)
    elif kind == RPAULI:
        Q = S.clone()
        for q in range(n):
            if strings[q0][q]:
                _pauli(Q, n, q, int(strings[q0][q]))
        S *= math.cos(t / 2)
        S.add_(Q, alpha=1j * math.sin(t / 2))
    else:
        hi, lo = max(q0, q1), min(q0, q1)
        v = S.view(S.shape[0], 2 ** (n - 1 - hi), 2, 2 ** (hi - lo - 1), 2, 2 ** lo)
        if kind == CZ:
            v[:, :, 1, :, 1] *= -1
            return
        ctl = v[:, :, 1] if q0 == hi else v[:, :, :, :, 1]     # (k, high, middle, 2, low) or (k, high, 2, middle, low)
        tdim = 3 if q0 == hi else 2
        ctl = ctl.movedim(tdim, 2)
        if kind == CNOT:
            a = ctl[:, :, 0].clone()
            ctl[:, :, 0] = ctl[:, :, 1]
            ctl[:, :, 1] = a
        else:
            _rotate(ctl, {CRX: RX, CRY: RY, CRZ: RZ}[kind], t)


def _generator(S, n, g, strings):
    """K S for the gate's generator K, a new tensor."""
    kind, q0, q1 = int(g[0]), int(g[1]), int(g[2])
    Q = S.clone()
    if kind == RPAULI:
        for q in range(n):
            if strings[q0][q]:
                _pauli(Q, n, q, int(strings[q0][q]))
    elif kind <= RZ:
        _pauli(Q, n, q0, kind + 1)
    else:
        _pauli(Q, n, q1, kind - CRX + 1)
        _bits(Q, n, q0)[:, :, 0] = 0
    return Q


def _exact_one(pr, case):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    n, gates, strings, P, theta = pr["n"], pr["gates"], pr["strings"], pr["P"], pr["theta"]
    rots = [i for i in range(len(gates)) if gates[i][3] >= 0]
    want_metric = case["op"] not in ("grad", "autograd")
    most = 27e9 if dev == "cuda" else 2e8
    stack = want_metric and (len(rots) + 1) * 2.0 ** n * 16 * (1 + len(rots) / 600) <= most
    if want_metric and not stack and case["op"] == "metric":
        return None
    dim = 2 ** n
    S = torch.zeros(len(rots) + 1 if stack else 1, dim, dtype=torch.complex128, device=dev)
    if pr["in_state"] is not None:
        S[0] = pr["in_state"].to(dev)
    else:
        S[0, 0] = 1
    k = 1
    for g in gates:
        t = theta[g[3]] if g[3] >= 0 else 0.0
        _apply(S[:k], n, g, t, strings)
        if stack and g[3] >= 0:
            S[k] = 0.5j * _generator(S[:1], n, g, strings)[0]
            k += 1
    out = {}
    J = np.zeros((len(rots), P))
    J[np.arange(len(rots)), [gates[i][3] for i in rots]] = 1.0
    if stack:
        M = torch.zeros(k, k, dtype=torch.complex128, device=dev)
        step = max(1, min(dim, 2 ** 28 // k // 16))
        for i in range(0, dim, step):
            X = S[:, i:i + step]
            M += X.conj() @ X.T.contiguous()
        M = M.cpu().numpy()
        T = M[0, 1:] @ J
        out["G"] = J.T @ M[1:, 1:] @ J - np.outer(T.conj(), T)
        out["T"] = T
    if case["op"] == "metric":
        return {"G": out["G"], "T": out["T"]}
    psi = S[:1].clone() if stack else S
    H = torch.zeros_like(psi)
    for letters, coeff in zip(pr["pauli"], pr["coeff"]):
        Q = psi.clone()
        for q in range(n):
            if letters[q]:
                _pauli(Q, n, q, int(letters[q]))
        H.add_(Q, alpha=float(coeff))
    out["E"] = float(torch.vdot(psi[0], H[0]).real)
    if stack:
        gr = 2.0 * (S[1:] @ H[0].conj()).real.cpu().numpy()
    else:
        gr = np.zeros(len(rots))
        both = torch.cat([H, psi])
        del H, psi, S
        for i in range(len(gates) - 1, -1, -1):
            g = gates[i]
            if g[3] >= 0:
                r = rots.index(i)
                gr[r] = -float(torch.vdot(both[0], _generator(both[1:], n, g, strings)[0]).imag)
            _apply(both, n, g, -theta[g[3]] if g[3] >= 0 else 0.0, strings)
    out["grad"] = gr @ J
    if case["op"] in ("grad", "autograd"):
        return {"E": out["E"], "grad": out["grad"]}
    dt, eps = _step_size(case)
    out["dtheta"] = np.linalg.solve(out["G"].real + eps * np.eye(P), -dt * out["grad"]) if stack else None
    if not case.get("want_G"):
        out.pop("G", None)
    elif not stack:
        out["G"] = None
    out.pop("T", None)
    if case["op"] in ("step_dev", "states"):
        out["status"] = None
    return out


def exact(case, seed):
    # a rotation per state: too slow beyond this
    prs = _problems(case, seed)
    if case["op"] == "batch":
        if sum(2.0 ** p["n"] * len(p["gates"]) ** 2 for p in prs) > 4e11:
            return None
        rs = [_exact_one(p, case) for p in prs]
        return {"dtheta": np.concatenate([r["dtheta"] for r in rs]), "grad": np.concatenate([r["grad"] for r in rs]),
                "E": np.asarray([r["E"] for r in rs])}
    return _exact_one(prs[0], case)
