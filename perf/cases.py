"""Timing cases of the simulator: what its users have it do, through its
public Python entry points, from 8-qubit calls to states of gigabytes.

A case is a dict of plain values; its "kind" names one of the paths below.
Which operators a case holds (how many, their target and control counts) is
fixed by the case; the qubits they act on, matrices, angles, observables and
states come from the seed.
"""
import math

import numpy as np
import torch

import paper_2311_01512_amd as qsim

DEV = "cuda"


# ---- the cases -------------------------------------------------------------------

def listed():
    return [
        # A small circuit run gate by gate with its norm and every qubit's outcome
        # probability read back: launches and call latency.
        {"name": "sv12_c128_ops", "kind": "sv_ops", "n": 12, "precision": "c128", "ops": 25, "probs": True},
        # One operator per call on a state of 4 GiB: 1- and 2-target gates with 0-3
        # controls, Pauli gadgets, swaps, Pauli tensors, phase gadgets.
        {"name": "sv28_c128_ops", "kind": "sv_ops", "n": 28, "precision": "c128", "ops": 14, "probs": False},
        # The large many-target workload: 5-target unitaries with 0-3 controls.
        {"name": "sv27_c64_dense5", "kind": "sv_dense", "n": 27, "precision": "c64", "ops": 4, "tmin": 5, "tmax": 5},
        # Many-target unitaries in double precision, 3 to 6 targets.
        {"name": "sv25_c128_dense3to6", "kind": "sv_dense", "n": 25, "precision": "c128", "ops": 4, "tmin": 3,
         "tmax": 6},
        # Noisy simulation, one operator per call: unitaries, Kraus maps, closed-form
        # channels and gadgets on a density matrix of 1 GiB.
        {"name": "dm13_c128_ops", "kind": "dm_ops", "n": 13, "precision": "c128", "ops": 14},
        # The headline workload: a recorded random circuit as run-time specialised tile
        # steps on 28 qubits.
        {"name": "circuit28_c64_tiles", "kind": "circuit", "n": 28, "precision": "c64", "ops": 250, "fuse": 13,
         "specialize": True},
        # A recorded circuit of moderate size in double precision, generic tile kernel.
        {"name": "circuit18_c128_tiles", "kind": "circuit", "n": 18, "precision": "c128", "ops": 200, "fuse": 11,
         "specialize": False},
        # A recorded noisy circuit on a density matrix, specialised tile steps.
        {"name": "dmcircuit12_c64_tiles", "kind": "dm_circuit", "n": 12, "precision": "c64", "ops": 100, "fuse": 12,
         "specialize": True},
        # Reading a large state: norm, outcome probabilities, a 20-term Pauli sum, an
        # inner product.
        {"name": "calc28_c64", "kind": "sv_calc", "n": 28, "precision": "c64", "terms": 20},
        # Reading a density matrix: trace, purity, outcome probability, Pauli sum and the
        # reduced state of half its qubits.
        {"name": "dmcalc13_c128", "kind": "dm_calc", "n": 13, "precision": "c128", "terms": 20, "traced": 6},
        # Batched variational circuits of uneven size: energies and all gradients.
        {"name": "batch192_c64_grads", "kind": "batch", "circuits": 192, "nmin": 10, "nmax": 20, "layers": 6,
         "terms": 20, "precision": "c64", "grads": True, "specialize": True},
        # Energy and adjoint gradient of one circuit with parametrised Pauli gadgets.
        {"name": "grad22_c128", "kind": "grad", "n": 22, "precision": "c128", "ops": 45, "terms": 20},
    ]


def draw(rng):
    kind = rng.choice(["sv_ops", "sv_dense", "dm_ops", "circuit", "dm_circuit", "sv_calc", "dm_calc", "batch", "grad"])
    prec = rng.choice(["c64", "c128"])
    c = {"kind": kind, "precision": prec}
    if kind == "sv_ops":
        c.update(n=rng.randint(8, 27), ops=rng.randint(5, 25), probs=rng.random() < 0.3)
    elif kind == "sv_dense":
        lo = rng.randint(3, 6)
        c.update(n=rng.randint(12, 25), ops=rng.randint(1, 5), tmin=lo, tmax=rng.randint(lo, 6))
    elif kind == "dm_ops":
        c.update(n=rng.randint(5, 12), ops=rng.randint(5, 20))
    elif kind in ("circuit", "dm_circuit"):
        dm = kind == "dm_circuit"
        c.update(n=rng.randint(6, 12) if dm else rng.randint(12, 26), ops=rng.randint(30, 200),
                 fuse=rng.randint(10, 13), specialize=rng.random() < 0.5)
    elif kind == "sv_calc":
        c.update(n=rng.randint(8, 27), terms=rng.randint(1, 40))
    elif kind == "dm_calc":
        n = rng.randint(5, 12)
        c.update(n=n, terms=rng.randint(1, 40), traced=rng.randint(1, n - 1))
    elif kind == "batch":
        lo = rng.randint(8, 13)
        c.update(circuits=rng.randint(4, 96), nmin=lo, nmax=lo + rng.randint(1, 6), layers=rng.randint(1, 6),
                 terms=rng.randint(5, 20), grads=rng.random() < 0.7, specialize=rng.random() < 0.3)
    else:
        c.update(n=rng.randint(10, 23), ops=rng.randint(10, 45), terms=rng.randint(1, 20))
    return c


# ---- operators and states -----------------------------------------------------------

def _haar(rng, rows, cols):
    """Haar-random matrix with orthonormal columns."""
    q, r = np.linalg.qr(rng.standard_normal((rows, cols)) + 1j * rng.standard_normal((rows, cols)))
    return q * (np.diagonal(r) / np.abs(np.diagonal(r)))


PAULI = np.array([[[1, 0], [0, 1]], [[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=complex)


def _depolarising(p):
    return np.sqrt([1 - p, p / 3, p / 3, p / 3])[:, None, None] * PAULI


def _depolarising2(p):
    return np.stack([np.sqrt(p / 15 if a or b else 1 - p) * np.kron(PAULI[a], PAULI[b])
                     for a in range(4) for b in range(4)])


def _dephasing(p):
    return np.sqrt([1 - p, p])[:, None, None] * PAULI[[0, 3]]


def _damping(p):
    return np.array([[[1, 0], [0, np.sqrt(1 - p)]], [[0, np.sqrt(p)], [0, 0]]], dtype=complex)


def _kraus2(rng):
    """Random two-qubit Kraus map of four operators."""
    return _haar(rng, 16, 4).reshape(4, 4, 4)


def _pauli_sum(rng, n, terms):
    return rng.integers(0, 4, size=(terms, n)).astype(np.int32), rng.standard_normal(terms)


def _ansatz(n, angles, layers):
    """Hardware-efficient ansatz: RY and RZ on every qubit, then a CZ ladder, per layer."""
    ops, k = [], 0
    for _ in range(layers):
        for code in (2, 3):
            for q in range(n):
                ops.append({"op": "gadget", "targs": (q,), "paulis": (code,), "theta": -0.5 * angles[k], "param": k,
                            "scale": -0.5})
                k += 1
        ops += [{"op": "unitary", "ctrls": (q,), "targs": (q + 1,), "matrix": PAULI[3]} for q in range(n - 1)]
    return ops


def _rng(case, seed):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, case.get("n", 0), case.get("ops", case.get("circuits", 0))])


def _pick(rng, n, k):
    return tuple(int(q) for q in rng.choice(n, size=k, replace=False))


def _unitary(rng, n, k, s):
    qs = _pick(rng, n, k + s)
    return {"op": "unitary", "targs": qs[:k], "ctrls": qs[k:], "matrix": _haar(rng, 1 << k, 1 << k)}


def _paulis(rng, n, kind):
    w = int(rng.integers(1, n + 1))
    targs = _pick(rng, n, w)
    paulis = tuple(int(p) for p in rng.integers(1, 4, size=w))
    return {"op": kind, "targs": targs, "paulis": paulis, "theta": float(rng.uniform(0, 2 * np.pi))}


SV_KINDS = ("gate1", "gate2", "gadget", "gate1", "swap", "gate2", "tensor", "gadget", "phase", "gate2")
DM_KINDS = ("gate1", "gate2", "depolarising", "damping", "kraus2", "dephasing", "gadget", "kraus1", "depolarising2")
CIRC_KINDS = ("gate1", "gate2", "gadget")
DM_CIRC_KINDS = ("gate1", "gate2", "kraus1", "damping_kraus", "kraus2")


def _make_op(rng, n, kind, i):
    if kind == "gate1":
        return _unitary(rng, n, 1, 0)
    if kind == "gate2":
        return _unitary(rng, n, 2, i % 4)
    if kind == "gadget":
        return _paulis(rng, n, "gadget")
    if kind == "tensor":
        return _paulis(rng, n, "pauli_tensor")
    if kind == "phase":
        op = _paulis(rng, n, "phase_gadget")
        op["paulis"] = (3,) * len(op["targs"])
        return op
    if kind == "swap":
        return {"op": "swap", "targs": _pick(rng, n, 2)}
    if kind == "kraus1":
        return {"op": "kraus", "targs": _pick(rng, n, 1), "kraus": _depolarising(rng.uniform(0, 0.05))}
    if kind == "damping_kraus":
        return {"op": "kraus", "targs": _pick(rng, n, 1), "kraus": _damping(rng.uniform(0, 0.1))}
    if kind == "kraus2":
        return {"op": "kraus", "targs": _pick(rng, n, 2), "kraus": _kraus2(rng)}
    k = 2 if kind.endswith("2") else 1
    return {"op": kind, "targs": _pick(rng, n, k), "p": float(rng.uniform(0, 0.05))}


def _kinds(case):
    table = {"sv_ops": SV_KINDS, "dm_ops": DM_KINDS, "circuit": CIRC_KINDS, "dm_circuit": DM_CIRC_KINDS}[case["kind"]]
    return [table[i % len(table)] for i in range(case["ops"])]


def _dm_ctrls(ops):
    """Density matrices: two-qubit unitaries without controls (as the noisy workload has them)."""
    for op in ops:
        if op["op"] == "unitary":
            op["ctrls"] = ()
    return ops


def _ops(case, rng):
    n = case["n"]
    if case["kind"] == "sv_dense":
        spread = case["tmax"] - case["tmin"] + 1
        return [_unitary(rng, n, case["tmin"] + i % spread, i % 4) for i in range(case["ops"])]
    if case["kind"] == "grad":
        ops, p = [], 0
        for i in range(case["ops"]):
            if i % 3 == 2:
                ops.append(_unitary(rng, n, 1 + (i // 3) % 2, (i // 6) % 2))
            else:
                op = _paulis(rng, n, "gadget")
                op.update(param=p, scale=-0.5)
                p += 1
                ops.append(op)
        return ops
    ops = [_make_op(rng, n, kind, i) for i, kind in enumerate(_kinds(case))]
    return _dm_ctrls(ops) if case["kind"].startswith("dm") else ops


def _params(ops):
    """Parameters of a gradient case: the angles that its gadgets were drawn with."""
    return np.array([op["theta"] / op["scale"] for op in ops if "param" in op])


def _dtype(case):
    return torch.complex64 if case["precision"] == "c64" else torch.complex128


def _state(case, seed, salt=0):
    """A normalised random statevector, or the projector on one as a Choi vector."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (int(seed) + 17 * salt) + case["n"])
    a = torch.randn(1 << case["n"], dtype=_dtype(case), device=DEV, generator=g)
    a /= torch.linalg.vector_norm(a)
    if not case["kind"].startswith("dm"):
        return a
    return (a.conj()[:, None] * a[None, :]).reshape(-1)   # entry j + k 2^n = a_j conj(a_k)


def _qureg(case, amps):
    q = qsim.Qureg(case["n"], density=case["kind"].startswith("dm"), precision=case["precision"])
    q.tensor.copy_(amps)
    return q


def _apply(q, op):
    kind = op["op"]
    if kind == "depolarising":
        q.apply_depolarising(op["targs"][0], op["p"])
    elif kind == "damping":
        q.apply_damping(op["targs"][0], op["p"])
    elif kind == "dephasing":
        q.apply_dephasing(op["targs"][0], op["p"])
    elif kind == "depolarising2":
        q.apply_two_qubit_depolarising(op["targs"][0], op["targs"][1], op["p"])
    else:
        q.run_ops([op])


def _batch_sizes(case):
    lo, hi = case["nmin"], case["nmax"]
    return [lo + (7 * c) % (hi - lo + 1) for c in range(case["circuits"])]


def _batch_inputs(case, seed):
    rng = _rng(case, seed)
    out = []
    for n in _batch_sizes(case):
        angles = rng.uniform(0, 2 * np.pi, size=2 * n * case["layers"])
        codes, coeffs = _pauli_sum(rng, n, case["terms"])
        out.append((n, angles, codes, coeffs))
    return out


# ---- one pass --------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        inputs = _batch_inputs(case, seed)
        b = qsim.Batch(precision=case["precision"])
        for n, angles, codes, coeffs in inputs:
            b.add_circuit(n, _ansatz(n, angles, case["layers"]), angles.size, codes, coeffs)
        b.compile()
        if case["specialize"]:
            b.specialize()
        return {"case": case, "batch": b, "params": np.concatenate([a for _, a, _, _ in inputs])}
    rng = _rng(case, seed)
    s = {"case": case, "q": _qureg(case, _state(case, seed))}
    if kind in ("sv_calc", "dm_calc"):
        s["sum"] = _pauli_sum(rng, case["n"], case["terms"])
        s["qubits"] = _pick(rng, case["n"], 3)
        if kind == "sv_calc":
            s["other"] = _qureg(case, _state(case, seed, salt=1))
        else:
            s["traced"] = sorted(_pick(rng, case["n"], case["traced"]))
            s["reduced"] = qsim.Qureg(case["n"] - case["traced"], density=True, precision=case["precision"])
        return s
    s["ops"] = _ops(case, rng)
    if kind in ("circuit", "dm_circuit"):
        s["circuit"] = qsim.Circuit(case["n"], s["ops"], density=kind == "dm_circuit")
        s["circuit"].compile(case["fuse"], case["precision"])
        if case["specialize"]:
            s["circuit"].specialize()
    elif kind == "grad":
        s["circuit"] = qsim.Circuit(case["n"], s["ops"])
        s["lam"] = qsim.Qureg(case["n"], precision=case["precision"])
        s["params"] = _params(s["ops"])
        s["sum"] = _pauli_sum(rng, case["n"], case["terms"])
    return s


def _values(case, v):
    """Scalars read from a state, in the precision that the state is held in."""
    return np.asarray(v, dtype=np.float32 if case["precision"] == "c64" else np.float64)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        e, g = s["batch"].run(s["params"], grads=case["grads"])
        return {"energies": _values(case, e), "grads": _values(case, g)} if case["grads"] else _values(case, e)
    q = s["q"]
    if kind in ("sv_ops", "sv_dense", "dm_ops"):
        for op in s["ops"]:
            _apply(q, op)
        if not case.get("probs"):
            return q.tensor
        return {"state": q.tensor, "probs": _values(case, [q.total_prob()] + [q.prob_of_outcome(k, 0)
                                                                             for k in range(case["n"])])}
    if kind in ("circuit", "dm_circuit"):
        s["circuit"].apply(q)
        return q.tensor
    if kind == "sv_calc":
        z = q.inner_product(s["other"])
        return {"probs": _values(case, [q.total_prob()] + [q.prob_of_outcome(k, 1) for k in s["qubits"]]),
                "expec": _values(case, [q.expec_pauli_sum(*s["sum"]).real]), "inner": _values(case, [z.real, z.imag])}
    if kind == "dm_calc":
        q.partial_trace(s["traced"], out=s["reduced"])
        return {"reduced": s["reduced"].tensor, "expec": _values(case, [q.expec_pauli_sum(*s["sum"]).real]),
                "scalars": _values(case, [q.trace().real, q.purity().real] +
                                   [q.prob_of_outcome(k, 0) for k in s["qubits"]])}
    s["circuit"].set_params(s["params"])
    e, g = s["circuit"].adjoint_gradient(q, s["lam"], *s["sum"])
    return {"energy": _values(case, [e]), "grads": _values(case, g), "psi": q.tensor}


# ---- what a pass cannot do without ----------------------------------------------------------

def _op_share(op_kind, i, density):
    """Share of the state that an operator has to read and write."""
    if op_kind == "gate2":
        return 1.0 if density else 0.5 ** (i % 4)
    return {"swap": 0.5, "dephasing": 0.5}.get(op_kind, 1.0)


_OP_FLOPS = {"gate1": 16, "gate2": 32, "gadget": 12, "phase": 6, "tensor": 0, "swap": 0, "kraus1": 32, "kraus2": 128,
             "damping_kraus": 32, "depolarising": 6, "damping": 4, "dephasing": 2, "depolarising2": 6}


def _op_flops(op_kind, density):
    f = _OP_FLOPS[op_kind]
    return 2 * f if density and op_kind in ("gate1", "gate2", "gadget") else f


def work(case):
    kind = case["kind"]
    amp = 8 if case["precision"] == "c64" else 16
    if kind == "batch":
        # rotations on phi (and, with gradients, back on phi and lambda with their products)
        per_rot, per_term = (6 * 3 + 4, 8) if case["grads"] else (6, 8)
        flops = sum((2.0 * n * case["layers"] * per_rot + case["terms"] * per_term) * (1 << n)
                    for n in _batch_sizes(case))
        params = sum(2 * n * case["layers"] for n in _batch_sizes(case))
        return {"bytes": 8.0 * params * (2 if case["grads"] else 1), "flops": flops}
    dm = kind.startswith("dm")
    num = float(1 << (2 * case["n"] if dm else case["n"]))
    if kind in ("sv_ops", "dm_ops"):
        b = sum(2 * amp * num * _op_share(k, i, dm) for i, k in enumerate(_kinds(case)))
        f = sum(num * _op_flops(k, dm) * _op_share(k, i, dm) for i, k in enumerate(_kinds(case)))
        if case.get("probs"):
            b += amp * num * (1 + case["n"] / 2)
        return {"bytes": b, "flops": f}
    if kind == "sv_dense":
        spread = case["tmax"] - case["tmin"] + 1
        share = [0.5 ** (i % 4) for i in range(case["ops"])]
        return {"bytes": sum(2 * amp * num * s for s in share),
                "flops": sum(8 * num * s * 2 ** (case["tmin"] + i % spread) for i, s in enumerate(share))}
    if kind in ("circuit", "dm_circuit"):
        return {"bytes": 2 * amp * num,
                "flops": sum(num * _op_flops(k, dm) * _op_share(k, i, dm) for i, k in enumerate(_kinds(case)))}
    if kind == "sv_calc":
        return {"bytes": amp * num * (1 + 1.5 + 1 + 2), "flops": num * (4 + 6 + 4 * case["terms"] + 8)}
    if kind == "dm_calc":
        kept = num / 2 ** case["traced"]
        diag = math.sqrt(num)
        return {"bytes": amp * (num + kept + kept / 2 ** case["traced"] + diag * (case["terms"] + 2.5)),
                "flops": 4 * num + 2 * kept + 8 * diag * case["terms"]}
    # gradient: forward, H psi, then back on both states with one product per parametrised gadget
    fixed = [1 + (i // 3) % 2 for i in range(case["ops"]) if i % 3 == 2]
    gadgets = case["ops"] - len(fixed)
    return {"bytes": 2 * amp * num * 3 * case["ops"],
            "flops": num * (gadgets * (3 * 12 + 8) + sum(3 * 8 * 2 ** k for k in fixed) + 8 * case["terms"])}


# ---- the same in 64 bits, in plain torch -----------------------------------------------------

def _bits_view(v, bits, qubits):
    """v (.., 2^bits) with a dimension of its own for each of the qubits, highest
    first; returns the view and each qubit's dimension."""
    shape, dims, top = list(v.shape[:-1]), {}, bits
    for q in sorted(qubits, reverse=True):
        shape += [1 << (top - q - 1), 2]
        dims[q] = len(shape) - 1
        top = q
    return v.view(shape + [1 << top]), dims


def _x_matrix(v, bits, ctrls, targs, m):
    """Controlled matrix on v in place; entries of m are numbers, or tensors
    that broadcast over the leading dimensions of v."""
    t, dims = _bits_view(v, bits, tuple(ctrls) + tuple(targs))
    d = 1 << len(targs)

    def part(i):
        index = [slice(None)] * t.dim()
        for c in ctrls:
            index[dims[c]] = 1
        for k, q in enumerate(targs):
            index[dims[q]] = (i >> k) & 1
        return t[tuple(index)]

    old = [part(i).clone() for i in range(d)]
    for r in range(d):
        acc = None
        for c in range(d):
            e = m[r][c]
            if isinstance(e, torch.Tensor):
                e = e.reshape(e.shape + (1,) * (old[c].dim() - e.dim()))
            elif e == 0:
                continue
            if acc is None:
                acc = old[c] * e
            elif isinstance(e, torch.Tensor):
                acc += old[c] * e
            else:
                acc.add_(old[c], alpha=e)
        if acc is None:
            part(r).zero_()
        else:
            part(r).copy_(acc)


def _signs(mask, bits):
    """(-1)^popcount(i & mask) for i < 2^bits."""
    s = torch.ones(1, dtype=torch.float64, device=DEV)
    for b in range(bits):
        s = torch.cat([s, -s if (mask >> b) & 1 else s])
    return s


def _x_pauli(v, bits, x, yz, ny):
    """The Pauli string with flip mask x and sign mask yz applied to v."""
    h = bits // 2
    lo = (1 << h) - 1
    w = v.view(1 << (bits - h), 1 << h) * _signs(yz & lo, h)
    w *= _signs(yz >> h, bits - h)[:, None]
    if x & lo:
        w = w[:, torch.arange(1 << h, device=DEV) ^ (x & lo)]
    if x >> h:
        w = w[torch.arange(1 << (bits - h), device=DEV) ^ (x >> h)]
    return w.reshape(-1) * (1, 1j, -1, -1j)[ny & 3]


def _masks(targs, paulis):
    x = sum(1 << t for t, p in zip(targs, paulis) if p in (1, 2))
    yz = sum(1 << t for t, p in zip(targs, paulis) if p in (2, 3))
    return x, yz, sum(1 for p in paulis if p == 2)


def _list_matrix(m):
    return [[complex(e) for e in row] for row in np.asarray(m)]


def _x_op(v, n, op, sign=1):
    """A statevector operator (its adjoint for sign = -1); returns the new vector."""
    kind = op["op"]
    if kind == "unitary":
        m = np.asarray(op["matrix"])
        _x_matrix(v, n, op["ctrls"], op["targs"], _list_matrix(m if sign > 0 else m.conj().T))
        return v
    if kind == "swap":
        _x_matrix(v, n, (), op["targs"], _list_matrix(np.eye(4)[[0, 2, 1, 3]]))
        return v
    p = _x_pauli(v, n, *_masks(op["targs"], op["paulis"]))
    if kind == "pauli_tensor":
        return p
    p *= 1j * sign * math.sin(op["theta"])
    return v.mul_(math.cos(op["theta"])).add_(p)


def _kraus_of(op):
    kind = op["op"]
    if kind == "unitary":
        return [op["matrix"]]
    if kind == "kraus":
        return op["kraus"]
    return {"depolarising": _depolarising, "damping": _damping,
            "dephasing": _dephasing, "depolarising2": _depolarising2}[kind](op["p"])


def _x_dm_op(v, n, op):
    """sum_m K_m rho K_m^dagger on the Choi vector (rows on bits 0..n-1)."""
    if op["op"] == "gadget":
        v = _x_op(v, 2 * n, op)
        _, _, ny = _masks(op["targs"], op["paulis"])
        cols = dict(op, targs=[t + n for t in op["targs"]], theta=(-1) ** (ny + 1) * op["theta"])
        return _x_op(v, 2 * n, cols)
    total = None
    for k in _kraus_of(op):
        w = v.clone()
        _x_matrix(w, 2 * n, (), op["targs"], _list_matrix(k))
        _x_matrix(w, 2 * n, (), [t + n for t in op["targs"]], _list_matrix(np.conj(k)))
        total = w if total is None else total.add_(w)
    return total


def _term_masks(codes):
    return _masks(range(len(codes)), [int(c) for c in codes])


def _x_hamiltonian(v, n, codes, coeffs):
    out = torch.zeros_like(v)
    for code, h in zip(codes, coeffs):
        out.add_(_x_pauli(v, n, *_term_masks(code)), alpha=float(h))
    return out


def _x_batch(case, seed):
    """Energies and gradients; circuits of one size run side by side."""
    inputs = _batch_inputs(case, seed)
    energies, grads = [None] * len(inputs), [None] * len(inputs)
    paulis = {2: [[0, -1j], [1j, 0]], 3: [[1, 0], [0, -1]]}
    for n in sorted(set(i[0] for i in inputs)):
        at = [c for c, i in enumerate(inputs) if i[0] == n]
        ang = torch.tensor(np.stack([inputs[c][1] for c in at]), device=DEV)
        cos, sin = torch.cos(ang / 2).to(torch.complex128), torch.sin(ang / 2).to(torch.complex128)
        z = torch.zeros(len(at), dtype=torch.complex128, device=DEV)
        ladder = torch.ones(1 << n, dtype=torch.float64, device=DEV)
        for q in range(n - 1):
            index = torch.arange(1 << n, device=DEV)
            ladder = torch.where(((index >> q) & 3) == 3, -ladder, ladder)

        def rotation(v, q, code, k, sign):   # exp(-i sign angle P / 2)
            c, s = cos[:, k], sign * sin[:, k]
            _x_matrix(v, n, (), (q,), [[c, -s], [s, c]] if code == 2 else [[c - 1j * s, z], [z, c + 1j * s]])

        plan, k = [], 0
        for _ in range(case["layers"]):
            for code in (2, 3):
                for q in range(n):
                    plan.append((q, code, k))
                    k += 1
            plan.append(None)
        v = torch.zeros(len(at), 1 << n, dtype=torch.complex128, device=DEV)
        v[:, 0] = 1
        for step in plan:
            if step is None:
                v *= ladder
            else:
                rotation(v, *step, 1)
        lam = torch.stack([_x_hamiltonian(v[j], n, inputs[c][2], inputs[c][3]) for j, c in enumerate(at)])
        e = (v.conj() * lam).sum(1).real
        g = torch.zeros(len(at), k, dtype=torch.float64, device=DEV)
        if case["grads"]:
            for step in reversed(plan):
                if step is None:
                    v *= ladder
                    lam *= ladder
                    continue
                q, code, k = step
                p = v.clone()
                _x_matrix(p, n, (), (q,), paulis[code])
                g[:, k] = (lam.conj() * p).sum(1).imag
                rotation(v, q, code, k, -1)
                rotation(lam, q, code, k, -1)
        for j, c in enumerate(at):
            energies[c], grads[c] = float(e[j]), g[j].cpu().numpy()
    e = np.array(energies)
    return {"energies": e, "grads": np.concatenate(grads)} if case["grads"] else e


def _prob(v, bits, q, outcome):
    t, dims = _bits_view(v, bits, (q,))
    return float(t.select(dims[q], outcome).abs().square().sum())


def exact(case, seed):
    kind, n = case["kind"], case.get("n")
    if kind == "batch":
        return _x_batch(case, seed)
    rng = _rng(case, seed)
    v = _state(case, seed).to(torch.complex128)
    if kind in ("sv_calc", "dm_calc"):
        codes, coeffs = _pauli_sum(rng, n, case["terms"])
        qubits = _pick(rng, n, 3)
        if kind == "sv_calc":
            w = _state(case, seed, salt=1).to(torch.complex128)
            e = sum(float(h) * float(torch.vdot(v, _x_pauli(v, n, *_term_masks(c))).real) for c, h in zip(codes, coeffs))
            z = complex(torch.vdot(v, w))
            return {"probs": np.array([float(v.abs().square().sum())] + [_prob(v, n, q, 1) for q in qubits]),
                    "expec": np.array([e]), "inner": np.array([z.real, z.imag])}
        traced = sorted(_pick(rng, n, case["traced"]))
        rho = v.view(1 << n, 1 << n)   # [column][row]
        k = torch.arange(1 << n, device=DEV)
        e = 0.0
        for c, h in zip(codes, coeffs):
            x, yz, ny = _term_masks(c)
            # P[l][k] = i^ny (-1)^popc(k & yz) for l = k ^ x; Tr(P rho) = sum_k P[k ^ x][k] rho[k][k ^ x]
            e += float(h) * float(((rho[k ^ x, k] * _signs(yz, n)).sum() * (1, 1j, -1, -1j)[ny & 3]).real)
        diag = rho[k, k].real
        t, dims = _bits_view(v, 2 * n, [q for q in traced] + [q + n for q in traced])
        red = None
        for i in range(1 << len(traced)):
            index = [slice(None)] * t.dim()
            for j, q in enumerate(traced):
                index[dims[q]] = index[dims[q + n]] = (i >> j) & 1
            red = t[tuple(index)].clone() if red is None else red.add_(t[tuple(index)])
        probs = [float(diag[((k >> q) & 1) == 0].sum()) for q in qubits]
        return {"reduced": red.reshape(-1), "expec": np.array([e]),
                "scalars": np.array([float(diag.sum()), float((rho * rho.T).sum().real)] + probs)}
    ops = _ops(case, rng)
    if kind in ("dm_ops", "dm_circuit"):
        for op in ops:
            v = _x_dm_op(v, n, op)
        return v
    for op in ops:
        v = _x_op(v, n, op)
    if kind != "grad":
        if not case.get("probs"):
            return v
        return {"state": v, "probs": np.array([float(v.abs().square().sum())] + [_prob(v, n, k, 0) for k in range(n)])}
    codes, coeffs = _pauli_sum(rng, n, case["terms"])
    lam = _x_hamiltonian(v, n, codes, coeffs)
    e, g = float(torch.vdot(v, lam).real), np.zeros(_params(ops).size)
    for op in reversed(ops):
        if "param" in op:
            p = _x_pauli(v, n, *_masks(op["targs"], op["paulis"]))
            g[op["param"]] += -2.0 * op["scale"] * float(torch.vdot(lam, p).imag)
        v = _x_op(v, n, op, -1)
        lam = _x_op(lam, n, op, -1)
    return {"energy": np.array([e]), "grads": g, "psi": v}
