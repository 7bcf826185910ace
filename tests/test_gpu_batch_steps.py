"""GPU parity of the level path's steps (sweeps of several blocks of a circuit)
where their form changes: the smallest level state, one and two tiles a
workgroup and more, programs of one block, of one step and of many, blocks of
1 to 5 qubits on neighbouring and scattered qubits."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _circuits(n):
    top = n - 1
    scattered = [W.Gate("h", (q,), ()) for q in range(n)]
    scattered += [W.Gate("cx", (q, top - q), ()) for q in range(n // 2)] + W.brickwork(n, 3, n)
    return [
        [W.Gate("u3", (top,), (0.7, 0.2, 0.4))],                                   # one block of one qubit
        [W.Gate("h", (0,), ()), W.Gate("cx", (0, top), ())],                        # one block, lowest to highest
        [W.Gate("u3", (q,), (0.1 + q, 0.2, 0.3)) for q in range(8)],                # one step of two blocks
        scattered,
    ]


@pytest.mark.parametrize("n", [13, 14, 17, 20])
def test_level_steps_match_oracle(n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    circuits = _circuits(n)
    masks = [1, 1 << (n - 1), 3 << (n - 2), (1 << n) - 1, 1 << (n // 2)]
    h = P.Handle()
    h.set_batch_level_qubits(13)
    b = P.Batch(h, [n] * len(circuits), circuits, [masks] * len(circuits), max_fused_qubits=5)
    exps, _, _ = b.run()
    for i, g in enumerate(circuits):
        ref, got = oracle.run(n, g), b.state(i).astype(np.complex128)
        # per block of a circuit (at most 3 n): 32 products of complex64
        assert np.linalg.norm(got - ref) <= 3 * n * 32 * 2.0 ** -24
        p = np.abs(got) ** 2
        idx = np.arange(1 << n, dtype=np.uint64)
        for e, m in zip(exps[i], masks):
            sign = 1.0 - 2.0 * (np.bitwise_count(idx & np.uint64(m)) & 1)
            # the sums and the norm are FP64: a few hundred roundings of terms
            # that add up to 1
            assert abs(e - np.sum(p * sign) / np.sum(p)) <= 512 * 2.0 ** -53
    b.close()
    h.close()
