"""The adjoint sweep as tile steps against a sweep written with the oracle,
operator by operator: the sizes where the path begins and where a state is
one tile, gates that fit no tile, more parametrised gadgets than a step takes,
angles whose cosine is not factored out, matrices that are not unitary (the
operator-by-operator sweep), and the plan kept between calls."""
import threading

import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qs():
    import paper_2311_01512_amd as pkg
    return pkg


def apply_h(psi, codes, coeffs):
    out = np.zeros_like(psi)
    for code, h in zip(codes, coeffs):
        out += h * oracle.apply_pauli_tensor(psi.copy(), list(range(len(code))), [int(c) for c in code])
    return out


def reference(psi, ops, codes, coeffs, num_params):
    """(energy, gradient) by the sweep that the entry point defines."""
    psi = oracle.run_ops(psi.copy(), ops)
    lam = apply_h(psi, codes, coeffs)
    e, g = np.vdot(psi, lam).real, np.zeros(num_params)
    for op in reversed(ops):
        if "param" in op:
            p = oracle.apply_pauli_tensor(psi.copy(), op["targs"], op["paulis"])
            g[op["param"]] += -2.0 * op["scale"] * np.vdot(lam, p).imag
        back = dict(op)
        if op["op"] == "gadget":
            back["theta"] = -op["theta"]
        else:
            back["matrix"] = op["matrix"].conj().T
        psi, lam = oracle.run_ops(psi, [back]), oracle.run_ops(lam, [back])
    return e, g


def gadget(rng, n, w, param, paulis=(1, 2, 3), theta=None):
    return {"op": "gadget", "targs": tuple(int(x) for x in rng.permutation(n)[:w]),
            "paulis": tuple(int(x) for x in rng.choice(paulis, size=w)), "param": param,
            "scale": float(rng.choice([1.0, -0.5])), "theta": theta}


def unitary(rng, n, k, nc, matrix=None):
    q = [int(x) for x in rng.permutation(n)[:k + nc]]
    return {"op": "unitary", "targs": tuple(q[:k]), "ctrls": tuple(q[k:]),
            "matrix": synth.haar_unitary(rng, 1 << k) if matrix is None else matrix}


def set_angles(ops, params):
    for op in ops:
        if "param" in op:
            op["theta"] = op["scale"] * params[op["param"]]


def check(qs, prec, n, ops, params, rng, terms=5, circuit=None):
    set_angles(ops, params)
    codes, coeffs = synth.random_pauli_sum(rng, n, terms)
    c = circuit or qs.Circuit(n, ops)
    c.set_params(params)
    start = synth.random_state(rng, 1 << n)
    psi, lam = qs.Qureg(n, precision=prec).set_amps(start), qs.Qureg(n, precision=prec)
    e, g = c.adjoint_gradient(psi, lam, codes, coeffs, num_params=len(params))
    if prec == "c64":
        start = start.astype(np.complex64).astype(np.complex128)
    we, wg = reference(start, ops, codes, coeffs, len(params))
    hnorm = max(1.0, np.abs(coeffs).sum())
    assert abs(e - we) < TOL[prec] * hnorm
    assert np.abs(g - wg).max() < (1e-10 * hnorm if prec == "c128" else 1e-4 * max(1.0, np.abs(wg).max()))
    return psi, start, c


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n", [3, 8, 9, 11, 12, 14])
def test_sizes(qs, prec, n):
    banner(f"adjoint tiles n={n} {prec}")
    rng = np.random.default_rng(8100 + n)
    ops = []
    for k in range(12):
        ops.append(gadget(rng, n, int(rng.integers(1, n + 1)), k % 9))
        ops.append(unitary(rng, n, 1 + k % 3 if n > 3 else 1, k % 2 + (k == 5 and n > 8)))
    psi, start, _ = check(qs, prec, n, ops, rng.uniform(0, 2 * np.pi, 9), rng)
    assert np.abs(psi.get_amps() - start).max() < TOL[prec]


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_operators_outside_tiles(qs, prec):
    """Gates of 4-6 targets and of 5 controls between the steps; an identity
    gadget; angles at and next to pi / 2."""
    rng = np.random.default_rng(8200)
    n, ops = 12, []
    for k, (nt, nc) in enumerate([(5, 0), (1, 5), (4, 1), (6, 2), (2, 4), (3, 0)]):
        ops.append(gadget(rng, n, 1 + k, k))
        ops.append(unitary(rng, n, nt, nc))
    ops.append({"op": "gadget", "targs": (4, 7), "paulis": (0, 0), "param": 6, "scale": 1.0, "theta": None})
    params = rng.uniform(0, 2 * np.pi, 7)
    params[1], params[3] = np.pi / 2 / ops[2]["scale"], (np.pi / 2 + 1e-3) / ops[6]["scale"]
    check(qs, prec, n, ops, params, rng)


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_many_commuting_gadgets(qs, prec):
    """70 commuting Z strings: more than one step's worth of sums."""
    rng = np.random.default_rng(8300)
    n = 10
    ops = [unitary(rng, n, 1, 0) for _ in range(6)] + [gadget(rng, n, 1 + k % 4, k, paulis=(3,)) for k in range(70)]
    ops += [gadget(rng, n, 2, 70 + k, paulis=(1, 2)) for k in range(5)]
    check(qs, prec, n, ops, rng.uniform(0, 2 * np.pi, 75), rng)


def test_matrices_that_are_not_unitary(qs):
    rng = np.random.default_rng(8400)
    n, ops = 10, []
    for k in range(6):
        ops.append(gadget(rng, n, 3, k))
        ops.append(unitary(rng, n, 2, 0, synth.random_matrix(rng, 4) / 3))
    check(qs, "c128", n, ops, rng.uniform(0, 2 * np.pi, 6), rng)


def test_kept_plan(qs):
    """New angles, appended operators, the other precision, and concurrent
    sweeps of one circuit on states of their own."""
    rng = np.random.default_rng(8500)
    n = 10
    ops = [op for k in range(5) for op in (gadget(rng, n, 1 + k, k), unitary(rng, n, 2, 1))]
    params = rng.uniform(0, 2 * np.pi, 6)
    c = None
    for _ in range(3):
        _, _, c = check(qs, "c128", n, ops, params, rng, circuit=c)
        params = rng.uniform(0, 2 * np.pi, 6)
    more = gadget(rng, n, 4, 5)
    more["theta"] = 0.1
    ops.append(more)
    c.add(more)
    check(qs, "c128", n, ops, params, rng, circuit=c)
    check(qs, "c64", n, ops, params, rng, circuit=c)
    codes, coeffs = synth.random_pauli_sum(rng, n, 4)
    starts = [synth.random_state(rng, 1 << n) for _ in range(4)]
    got = [None] * 4

    def sweep(i):
        import torch
        s = torch.cuda.Stream()
        psi, lam = (qs.Qureg(n, precision="c128", stream=s) for _ in range(2))
        psi.set_amps(starts[i])
        got[i] = [c.adjoint_gradient(psi, lam, codes, coeffs, num_params=6) for _ in range(5)]

    threads = [threading.Thread(target=sweep, args=(i,)) for i in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    for i in range(4):
        we, wg = reference(starts[i], ops, codes, coeffs, 6)
        for e, g in got[i]:
            assert abs(e - we) < 1e-11 and np.abs(g - wg).max() < 1e-10 * max(1.0, np.abs(coeffs).sum())
