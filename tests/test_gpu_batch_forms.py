"""Batched rotations with their factor taken out: angles where the form
changes (|cos| = |sin|) or a cosine or sine vanishes, segments (more rotations
on a few qubits than a segment takes, with fixed gates and CZs between), and the
observable's real and imaginary terms, on sizes around the paths' limits
(8: one operator per LDS pass; 9: one full wavefront; 10: four amplitudes per
thread; 13: several tiles), generic and specialised, against the oracle."""
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


ANGLES = np.array([0.0, np.pi / 2, np.pi, -np.pi / 2, 3 * np.pi / 2, np.pi / 4, np.nextafter(np.pi / 4, 1),
                   -np.pi / 4, 3 * np.pi / 4, 1e-9, np.pi / 2 + 1e-9, 20.5 * np.pi, 0.3, 2.2])


def problem(rng, n):
    """Two circuits' worth of rotations: every special angle, and a run of 90
    on three qubits."""
    ops, params = [], []

    def rotation(q, p, a):
        ops.append({"op": "gadget", "targs": (int(q),), "paulis": (int(p),), "param": len(params), "scale": 1.0,
                    "theta": float(a)})
        params.append(float(a))

    z = synth.pauli_matrix_2x2(3)
    for q in range(n):
        rotation(q, 2, rng.uniform(0, 6))
    for k, a in enumerate(ANGLES):
        rotation(rng.integers(n), 1 + k % 3, a)
        q = [int(x) for x in rng.permutation(n)[:2]]
        ops.append({"op": "unitary", "ctrls": (q[0],), "targs": (q[1],), "matrix": z})
    for k in range(90):
        rotation(k % min(3, n), 1 + k % 2, rng.choice(ANGLES) if k % 4 else rng.uniform(0, 6))
        if k % 30 == 7:
            ops.append({"op": "unitary", "ctrls": (), "targs": (k % n,), "matrix": synth.haar_unitary(rng, 2)})
    codes, coeffs = synth.random_pauli_sum(rng, n, 9)
    return ops, np.array(params), codes, coeffs


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_rotation_forms(qs, prec):
    rng = np.random.default_rng(6100)
    sizes = [3, 8, 9, 10, 11, 13]
    b = qs.Batch(precision=prec)
    problems = [problem(rng, n) for n in sizes]
    for n, (ops, params, codes, coeffs) in zip(sizes, problems):
        b.add_circuit(n, ops, len(params), codes, coeffs)
    b.compile()
    params = np.concatenate([p for _, p, _, _ in problems])
    want = [(oracle.sv_expec_pauli_sum(oracle.run_ops(oracle.zero_state(n), ops), codes, coeffs).real,
             oracle.param_shift_gradient(n, ops, codes, coeffs, len(p)))
            for n, (ops, p, codes, coeffs) in zip(sizes, problems)]
    for kind in ("generic", "specialised"):
        banner(f"batch rotation forms {prec} {kind}")
        if kind == "specialised":
            b.specialize()
        e, g = b.run(params)
        at = 0
        for k, (n, (_, p, _, coeffs)) in enumerate(zip(sizes, problems)):
            hnorm = max(1.0, np.abs(coeffs).sum())
            assert abs(e[k] - want[k][0]) < TOL[prec] * hnorm, (kind, n)
            bound = 1e-10 * hnorm if prec == "c128" else 1e-4 * max(1.0, np.abs(want[k][1]).max())
            assert np.abs(g[at:at + len(p)] - want[k][1]).max() < bound, (kind, n)
            at += len(p)
        e2, none = b.run(params, grads=False)
        assert none is None and np.array_equal(e, e2)
        for k, (n, (ops, _, _, _)) in enumerate(zip(sizes, problems)):
            psi = oracle.run_ops(oracle.zero_state(n), ops)
            assert np.abs(b.state(k) - psi).max() < TOL[prec] * np.abs(psi).max()
