"""GPU parity of Pauli expectations whose X/Y masks share sweeps: numbers of
masks around the five of one sweep, masks in each other's span, masks on the
lowest and highest qubits only, several terms on one mask, small states."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    return P


def _terms(n, kind, count, rng):
    if kind == "random":
        return W.random_pauli_terms(n, count, rng)
    if kind == "span":  # products of three strings: at most seven X/Y masks, in one span
        base = [rng.integers(0, 2, size=n) for _ in range(3)]
        out = []
        while len(out) < count:
            x = sum(b * int(rng.integers(0, 2)) for b in base) % 2
            z = rng.integers(0, 2, size=n)
            t = [(q, "IXZY"[int(x[q] + 2 * z[q])]) for q in range(n) if x[q] or z[q]]
            if t:
                out.append(t)
        return out
    # pairs of neighbours at both ends: XX, YY, XY, YX and ZZ share masks
    out = []
    for q in (0, max(0, n - 2)):
        for a in ("XX", "YY", "XY", "YX", "ZZ"):
            out.append([(q, a[0]), (q + 1, a[1])] if n > 1 else [(0, a[0])])
    return out + [[(q, "X")] for q in range(min(n, count))]


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,kind,count", [(1, "ends", 1), (2, "random", 7), (3, "span", 9), (5, "ends", 5), (7, "random", 1),
                                          (9, "random", 4), (10, "random", 5), (11, "random", 6), (12, "span", 20),
                                          (13, "random", 16), (14, "ends", 14), (16, "random", 33), (22, "random", 6),
                                          (23, "random", 11), (23, "ends", 9)])
def test_shared_sweeps_match_the_oracle(P, dt, n, kind, count):
    # FP64 products and sums of the state's own amplitudes on both sides: the
    # sum of 2^n terms of total weight 1 is off by less than 1e-12
    rng = np.random.default_rng(100 * n + count)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    h = P.Handle()
    st = P.State(h, n, dt)
    host = psi.astype(np.complex64 if dt == "c64" else np.complex128)
    P.sv_copy_from_host(st.s, host)
    terms = _terms(n, kind, count, rng)
    got = st.expect(terms)
    ref = host.astype(np.complex128)
    want = np.array([oracle.expect_pauli(ref, t) for t in terms])
    assert np.max(np.abs(got - want)) <= 1e-12
    np.testing.assert_array_equal(got, st.expect(terms))
    # a term alone has the value it has among others, up to the sums' order
    for i in (0, len(terms) - 1):
        assert abs(st.expect([terms[i]])[0] - got[i]) <= 1e-12
    st.close()
    h.close()
