"""Dense gates of 4-6 targets on the matrix cores against the oracle, where
the kernel's work units end: fewer groups than a wavefront takes (the vector
kernel), exactly one tile, a few waves, and more tiles than the grid has waves
(the persistent walk), with the lowest, the highest and unordered targets."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, amp_err, banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qs():
    import paper_2311_01512_amd as pkg
    return pkg


# log2 of the number of groups: below a tile, one tile, one block, more than
# 2048 tiles (512 blocks of 4 waves) with k >= 5
@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("k,groups", [(k, g) for k in (4, 5, 6) for g in (3, 4, 6)] + [(4, 13), (5, 16), (6, 16)])
def test_dense_gate_parity(qs, prec, k, groups):
    N = k + groups
    rng = np.random.default_rng(9100 + 100 * k + groups)
    sets = [tuple(range(k)), tuple(range(N - 1, N - 1 - k, -1)), tuple(int(q) for q in rng.permutation(N)[:k])]
    for targs in sets if groups < 10 else sets[2:]:
        banner(f"dense k={k} groups=2^{groups} {prec} {targs}")
        M = synth.haar_unitary(rng, 1 << k)
        psi = synth.random_state(rng, 1 << N)
        q = qs.Qureg(N, precision=prec).set_amps(psi)
        q.apply_unitary((), targs, M)
        assert amp_err(q.get_amps(), oracle.apply_gate(psi.copy(), (), targs, M)) < TOL[prec]


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("k", [4, 5, 6])
@pytest.mark.parametrize("extra", [4, 5, 7])
def test_controlled_dense_blocks(qs, prec, k, extra):
    """Controls take groups away (16, 8 and fewer are left for extra = 4 with
    0, 1, 2 controls); applied directly and as a compiled dense block."""
    N = k + extra
    rng = np.random.default_rng(9700 + 10 * k + extra)
    psi = synth.random_state(rng, 1 << N)
    ops = []
    for nc in (0, 1, 2):
        qubits = [int(x) for x in rng.permutation(N)[:k + nc]]
        ops.append({"op": "unitary", "targs": tuple(qubits[:k]), "ctrls": tuple(qubits[k:]),
                    "matrix": synth.haar_unitary(rng, 1 << k)})
    banner(f"controlled dense k={k} N={N} {prec}")
    want = oracle.run_ops(psi.copy(), ops)
    q = qs.Qureg(N, precision=prec).set_amps(psi).run_ops(ops)
    assert amp_err(q.get_amps(), want) < TOL[prec]
    c = qs.Circuit(N, ops).compile(6, prec)
    q.set_amps(psi)
    c.apply(q)
    assert amp_err(q.get_amps(), want) < TOL[prec]
