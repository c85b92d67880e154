"""Generic tile steps with one block per tile, and with blocks that walk
several tiles whose bases follow by an addition over the pivots."""
import numpy as np
import pytest

import synth
import test_gpu_adjoint_tiles as adjoint
from gpu_helpers import TOL, amp_err, banner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qs():
    import paper_2311_01512_amd as pkg
    return pkg


# 13 dimensions: 512 (complex64) or 256 (complex128) resident blocks walk 2048
# and 512 tiles; below, one tile per block, from a single block on, down to
# blocks of less than a wavefront
@pytest.mark.parametrize("prec,width,n", [("c64", 13, 24), ("c128", 13, 22), ("c64", 12, 12), ("c64", 12, 22),
                                          ("c128", 11, 13), ("c128", 11, 21), ("c64", 8, 15), ("c128", 8, 14)])
def test_generic_steps(qs, prec, width, n):
    banner(f"tile walk {prec} width {width} N={n}")
    ops = synth.config2_circuit(num_qubits=n, num_gates=60, seed=8950 + n)
    a = qs.Qureg(n, precision=prec).init_hashed(11)
    b = qs.Qureg(n, precision=prec).init_hashed(11)
    qs.Circuit(n, ops).compile(width, prec).apply(a)
    b.run_ops(ops)
    # 60 operators on either side
    assert amp_err(a.get_amps(), b.get_amps()) <= 2 * TOL[prec]


def test_adjoint_walk(qs):
    """2^12 tiles of 2^11 amplitudes, 2048 blocks."""
    n, rng = 23, np.random.default_rng(8960)
    ops = []
    for k in range(4):
        ops.append(adjoint.gadget(rng, n, int(rng.integers(1, n + 1)), k))
        ops.append(adjoint.unitary(rng, n, 1 + k % 2, k % 2))
    adjoint.check(qs, "c128", n, ops, rng.uniform(0, 2 * np.pi, 4), rng, terms=3)
