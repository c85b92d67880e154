"""Scalars that follow short and long queues of operators: the result's word is
watched for a while, then the stream is waited for."""
import numpy as np
import pytest

from gpu_helpers import banner

pytestmark = pytest.mark.gpu


# 24 qubits: 40 gates take several milliseconds, far longer than the watch;
# one and several blocks, two states whose calls alternate
@pytest.mark.parametrize("n,gates", [(1, 0), (1, 3), (10, 1), (18, 5), (24, 40)])
def test_scalars_after_queued_gates(n, gates):
    import torch

    import paper_2311_01512_amd as qs
    banner(f"scalars N={n} gates={gates}")
    rng = np.random.default_rng(70 + n)
    a = qs.Qureg(n, precision="c128")
    b = qs.Qureg(n, precision="c128", stream=torch.cuda.Stream())
    a.init_zero()
    b.init_zero()
    p = 1.0         # probability of 0 at qubit 0
    for rep in range(6):
        for g in range(gates):
            a.apply_unitary([], [0], np.array([[0, 1], [1, 0]], dtype=complex))
            u = np.linalg.qr(rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2)))[0]
            b.apply_unitary([], [0], u)
            amp = u @ (amp if rep or g else np.array([1.0, 0.0]))
        if gates:
            p = abs(amp[0]) ** 2
        flips = gates * (rep + 1) % 2
        # each gate and each sum of 2^n squares rounds by a few 2^-53
        tol = 1e-13 * (1 + gates * 6)
        assert a.prob_of_outcome(0, flips) == 1.0
        assert abs(b.prob_of_outcome(0, 0) - p) <= tol
        assert a.prob_of_outcome(0, 1 - flips) == 0.0
        assert abs(b.total_prob() - 1.0) <= tol
        # <00..0|X^k|00..0> of the two states: an amplitude of b
        want = (amp[flips] if gates else 1.0)
        b.sync()
        assert abs(a.inner_product(b) - want) <= tol


def test_purity_of_one_block():
    import paper_2311_01512_amd as qs
    banner("purity of one block")
    for n in (1, 3, 5):
        q = qs.Qureg(n, density=True, precision="c128").init_zero()
        for _ in range(3):
            assert abs(q.purity() - 1.0) <= 1e-15
