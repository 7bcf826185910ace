"""GPU parity of the sweeps that apply several fused blocks to each tile, at
the sizes where their rules change: one-tile states (up to 13 qubits complex64,
12 complex128), in-order sweeps (below 22 qubits), reordered ones (from 22)."""
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


def _program(n, seed):
    """Gates whose fused blocks have 1 to 5 qubits, neighbouring and scattered."""
    gates = W.serving_circuit(n, 4, np.random.default_rng(seed)) + W.brickwork(n, 4, seed)
    if n > 3:  # blocks from the lowest to the highest qubit, which are not padded
        gates += [W.Gate("cx", (0, n - 1), ()), W.Gate("cz", (1, n - 2), ()), W.Gate("cx", (n - 1, 1), ())]
    return gates + [W.Gate("u3", (n - 1,), (0.3, 0.2, 0.1))]


def _run(P, n, dt, gates, mode):
    h = P.Handle()
    h.set_tile_mode(mode)
    st = P.State(h, n, dt)
    st.run(gates, max_fused_qubits=5)
    got = st.to_numpy()
    st.close()
    h.close()
    return got


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 6, 9, 11, 12, 13, 14, 15, 17, 21, 22, 23])
def test_sweeps_of_several_blocks(P, dt, n):
    # a forced tile variant takes every block on its own; below 22 qubits the
    # sweeps' arithmetic and order are the same, so the bits are too; from 22
    # qubits blocks that commute may change places: a few rounding errors per
    # block (unit roundoff u, about 30 blocks, of amplitudes of 2-norm 1)
    gates = _program(n, 10 + n)
    got = _run(P, n, dt, gates, P.SV_TILE_AUTO)
    alone = _run(P, n, dt, gates, P.SV_TILE_NARROW)
    if n < 22:
        np.testing.assert_array_equal(got, alone)
    else:
        u = 2.0 ** -24 if dt == "c64" else 2.0 ** -53
        d = np.linalg.norm(got.astype(np.complex128) - alone.astype(np.complex128))
        assert d <= 30 * 32 * u
    if n <= 17:
        ref = oracle.run(n, gates)
        if dt == "c128":
            assert np.max(np.abs(got - ref)) <= 1e-10
        else:
            assert oracle.fidelity(ref, got.astype(np.complex128)) >= 1.0 - 1e-5


@pytest.mark.parametrize("dt,n", [("c64", 13), ("c128", 12), ("c64", 16), ("c128", 16), ("c64", 22)])
def test_long_programs_and_block_ranges(P, dt, n):
    # more blocks than one sweep takes, applied whole, in ranges and from a
    # recorded graph
    gates = W.serving_circuit(n, 40 if n < 22 else 10, np.random.default_rng(n))
    h = P.Handle()
    st = P.State(h, n, dt)
    f = P.fuse(gates, 5)
    P.sv_apply_fused(st.s, f.f)
    whole = st.to_numpy()
    g = P.Graph(st, gates, 5)
    for _ in range(2):
        P.sv_set_basis_state(st.s, 0)
        g.launch()
        np.testing.assert_array_equal(st.to_numpy(), whole)
    g.close()
    P.sv_set_basis_state(st.s, 0)
    cuts = [0, 1, f.count // 3, f.count // 2, f.count]
    for a, b in zip(cuts[:-1], cuts[1:]):
        P.sv_apply_fused_range(st.s, f.f, a, b - a)
    parts = st.to_numpy()
    if n < 22:
        np.testing.assert_array_equal(parts, whole)
    else:
        assert oracle.fidelity(parts.astype(np.complex128), whole.astype(np.complex128)) >= 1.0 - 1e-5
    st.close()
    f.free()
    h.close()
