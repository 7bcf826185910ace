"""GPU parity of Pauli expectations of small states whose joint sweeps have
different numbers of masks (filled up to one number): numbers of masks that
five does not divide, masks of a small span, on few and on many qubits."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,count", [(2, 3), (4, 15), (5, 31), (6, 40), (12, 31), (16, 11), (22, 7)])
def test_sweeps_of_different_sizes_match_the_oracle(dt, n, count):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    rng = np.random.default_rng(n + count)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    h = P.Handle()
    st = P.State(h, n, dt)
    host = psi.astype(np.complex64 if dt == "c64" else np.complex128)
    P.sv_copy_from_host(st.s, host)
    low = min(n, 5)  # X on every set of the lowest qubits, and strings on all
    terms = [[(q, "XY"[int(rng.integers(0, 2))]) for q in range(low) if (m >> q) & 1] for m in range(1, 1 << low)][:count]
    terms += W.random_pauli_terms(n, 3, rng)
    got = st.expect(terms)
    want = np.array([oracle.expect_pauli(host.astype(np.complex128), t) for t in terms])
    # FP64 products and sums of total weight 1
    assert np.max(np.abs(got - want)) <= 1e-12
    np.testing.assert_array_equal(got, st.expect(terms))
    st.close()
    h.close()
