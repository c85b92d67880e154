"""Statevector Pauli sums on both sides of the size where tiles take over from
gathers, and where the gathers' launches change: one block, the first size
with four amplitudes per thread, several blocks, one and several launches'
worth of terms; and the readings whose sum one block takes."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import banner, scalar_tol

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qs():
    import paper_2311_01512_amd as pkg
    return pkg


# 8 MiB is 20 qubits in complex64 and 19 in complex128
@pytest.mark.parametrize("n,T,prec", [(n, T, p) for p in ("c64", "c128")
                                      for n, T in ((8, 1), (9, 64), (10, 65), (11, 130), (13, 7))] +
                         [(20, 12, "c64"), (21, 40, "c64"), (19, 12, "c128"), (20, 40, "c128")])
def test_pauli_sums(qs, n, T, prec):
    banner(f"Pauli sum N={n} T={T} {prec}")
    rng = np.random.default_rng(8800 + 100 * n + T)
    codes, coeffs = synth.random_pauli_sum(rng, n, T)
    if T > 3:
        codes[0] = 0                                     # identity
        codes[1] = rng.choice([0, 3], size=n)            # diagonal
        codes[2], codes[2, 1] = 0, 2                     # one Y on a low qubit
        codes[3], codes[3, n - 1] = 0, 1                 # one X on the highest
    psi = synth.random_state(rng, 1 << n)
    q = qs.Qureg(n, precision=prec).set_amps(psi)
    got = q.expec_pauli_sum(codes, coeffs)
    want = oracle.sv_expec_pauli_sum(psi, codes, coeffs)
    assert abs(got - want) < scalar_tol(prec, np.abs(coeffs).sum())
    assert got == q.expec_pauli_sum(codes, coeffs) and got.imag == 0


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 5, 12, 13, 14])
def test_sums_of_one_and_more_blocks(qs, n, prec):
    """2^13 amplitudes are the last sum of one block."""
    rng = np.random.default_rng(8900 + n)
    a, b = synth.random_state(rng, 1 << n), synth.random_state(rng, 1 << n)
    qa, qb = (qs.Qureg(n, precision=prec).set_amps(v) for v in (a, b))
    tol = scalar_tol(prec)
    assert abs(qa.total_prob() - 1) < tol
    assert abs(qa.inner_product(qb) - np.vdot(a, b)) < tol
    for k in (0, n - 1):
        for bit in (0, 1):
            assert abs(qa.prob_of_outcome(k, bit) - oracle.sv_prob_of_outcome(a, k, bit)) < tol


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("n,T", [(2, 3), (6, 5), (8, 25), (10, 24), (11, 26)])
def test_density_sums(qs, n, T, prec):
    """Terms in groups of four, the last one partial; more than one launch."""
    rng = np.random.default_rng(8950 + n)
    psi = synth.random_state(rng, 1 << n)
    rho = np.outer(psi.conj(), psi).reshape(-1)
    q = qs.Qureg(n, density=True, precision=prec).set_amps(rho)
    codes, coeffs = synth.random_pauli_sum(rng, n, T)
    tol = scalar_tol(prec, np.abs(coeffs).sum())
    assert abs(q.expec_pauli_sum(codes, coeffs) - oracle.dm_expec_pauli_sum(rho, codes, coeffs)) < tol
    assert abs(q.trace() - 1) < scalar_tol(prec) and abs(q.purity() - 1) < scalar_tol(prec)
    assert abs(q.prob_of_outcome(n - 1, 1) - oracle.dm_prob_of_outcome(rho, n - 1, 1)) < scalar_tol(prec)


# several tiles per block; terms that pair by register bits, by thread bits and
# not at all, alone and combined, with sums of real and of imaginary parts
@pytest.mark.parametrize("n,prec", [(24, "c64"), (25, "c64"), (23, "c128"), (24, "c128")])
def test_tile_sums_of_many_tiles(qs, n, prec):
    banner(f"tile sums N={n} {prec}")
    rng = np.random.default_rng(8900 + n)
    rows = [np.zeros(n, int), rng.choice([0, 3], size=n)]
    for q, c in ((0, 1), (3, 2), (2, 1)):
        row = rng.choice([0, 3], size=n)
        row[q] = c
        rows.append(row)
    masks = [rng.integers(0, 2, size=n) for _ in range(7)]
    for x in masks + [masks[0] ^ masks[1], masks[2] ^ masks[5] ^ masks[6]]:
        for _ in range(2):
            rows.append(np.where(x, rng.choice([1, 2], size=n), rng.choice([0, 3], size=n)))
    codes = np.array(rows)
    coeffs = rng.normal(size=len(rows))
    q = qs.Qureg(n, precision=prec).init_hashed(8901)
    psi = q.get_amps().astype(np.complex128)
    got = q.expec_pauli_sum(codes, coeffs)
    # a hashed state's terms are about 2^(-n/2): complex64 products round by
    # 2 2^-24 of sum |a_i a_j| <= 1
    tol = 2.0 ** -22 if prec == "c64" else 1e-12
    assert abs(got - oracle.sv_expec_pauli_sum(psi, codes, coeffs).real) <= tol * np.abs(coeffs).sum()
