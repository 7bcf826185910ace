"""The complex64 sweeps of 22 qubits and more multiply bf16 parts of matrices and
amplitudes.  Where FP32 products are as exact or more so they take these: blocks
of one real gate, amplitudes and matrix entries whose parts lose bits."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
N = 22
CHAIN = [W.Gate("cx", (q, q + 1), ()) for q in range(4)]  # makes one block of five qubits


def _run(x, gates, dt="c64", split=True):
    import torch
    import paper_2308_01999_amd as P
    h = P.Handle()
    h.set_tile_mode(P.SV_TILE_AUTO if split else P.SV_TILE_NARROW)
    t = torch.from_numpy(x.astype(np.complex64 if dt == "c64" else np.complex128)).cuda()
    st = P.State(h, N, dt, basis=None, tensor=t)
    f = P.fuse(gates, 5)
    assert [len(b[0]) for b in f.blocks()] == [5]
    P.sv_apply_fused(st.s, f.f)
    out = st.to_numpy()
    f.free()
    st.close()
    h.close()
    return out


def _amplitudes(seed, real):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal(1 << N) + (0 if real else 1j * rng.standard_normal(1 << N))
    return (x / np.linalg.norm(x)).astype(np.complex64)


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("qubits", [(0,), (1,), (2,), (3,), (4,), (0, 4), (1, 3), (0, 1, 2), (0, 1, 2, 3), (0, 1, 2, 3, 4)])
@pytest.mark.parametrize("real", [True, False])
def test_real_gates_are_as_exact_as_fp32(qubits, real):
    # against the complex128 sweep of the same amplitudes, 2^22 of them: the two mean
    # squares are known to about 2^-10
    x = _amplitudes(len(qubits), real)
    gates = CHAIN + [W.Gate("u3", (q,), (0.7 + 0.3 * q, 0.0, 0.0)) for q in qubits]
    exact = _run(x, gates, "c128")
    split, fp32 = (np.linalg.norm(_run(x, gates, split=m) - exact) for m in (True, False))
    assert 0.0 < split <= fp32 * (1 + 2.0 ** -9), (split, fp32)


@pytest.mark.parametrize("exponent", [-104, -116, 60])
def test_scaled_states_keep_their_digits(exponent):
    # amplitudes about 2^-11 of the scale, from where the parts lose bits down to
    # FP32's smallest normal numbers, and far above 1
    x = (_amplitudes(7, False) * np.float32(2.0) ** np.float32(exponent)).astype(np.complex64)
    gates = CHAIN + [W.Gate("u3", (q,), (0.7, 0.2 * q, 0.4)) for q in range(5)]
    exact = _run(x, gates, "c128")
    split, fp32 = (np.linalg.norm((_run(x, gates, split=m) - exact) * 2.0 ** -exponent) for m in (True, False))
    assert 0.0 < split <= fp32, (split, fp32)


def test_permuted_amplitudes_are_unchanged():
    # 0, 1 and sums with zeros are exact: of amplitudes of any size FP32 has
    rng = np.random.default_rng(3)
    size = 10.0 ** rng.uniform(-44.5, 38.4, size=(2, 1 << N))
    parts = (size * rng.choice([-1.0, 1.0], size=size.shape)).astype(np.float32)
    parts[:, :2] = np.finfo(np.float32).max, np.finfo(np.float32).smallest_subnormal
    x = parts[0] + 1j * parts[1]
    got = _run(x.astype(np.complex64), CHAIN)
    i = np.arange(1 << N)
    j = i.copy()
    for q in range(4):
        j = j ^ (((j >> q) & 1) << (q + 1))
    assert np.array_equal(got[j], x.astype(np.complex64))


@pytest.mark.parametrize("scale", [2.0 ** -116, 2.0 ** 126])
def test_matrix_entries_of_any_size(scale):
    # a dense block with such entries, on amplitudes that give results near 1
    import torch
    import paper_2308_01999_amd as P
    rng = np.random.default_rng(5)
    m = (rng.standard_normal((32, 32)) + 1j * rng.standard_normal((32, 32))) / 8 * scale
    x = (rng.standard_normal(1 << N) + 1j * rng.standard_normal(1 << N)) / scale
    x = x.astype(np.complex64)

    def run(dt, mode):
        h = P.Handle()
        h.set_tile_mode(mode)
        t = torch.from_numpy(x.astype(np.complex64 if dt == "c64" else np.complex128)).cuda()
        st = P.State(h, N, dt, basis=None, tensor=t)
        f = P.Fused(P.sv_fuse_gates([((0, 2, 4, 6, 8), m, (), None)], 5))
        P.sv_apply_fused(st.s, f.f)
        out = st.to_numpy()
        f.free()
        st.close()
        h.close()
        return out

    exact = run("c128", P.SV_TILE_AUTO)
    split, fp32 = (np.linalg.norm(run("c64", k) - exact) for k in (P.SV_TILE_AUTO, P.SV_TILE_NARROW))
    assert 0.0 < split <= fp32, (split, fp32)


@pytest.mark.parametrize("qubits", [(2,), (0, 1, 2, 3, 4)])
@pytest.mark.parametrize("exponent", [0, -104])
def test_coupled_blocks_on_fp32_products(qubits, exponent):
    # a coupled block that takes FP32 products (one real gate), or whose amplitudes'
    # parts lose bits, or both: phases from outside the tile and from inside it
    import torch
    import paper_2308_01999_amd as P
    x = (_amplitudes(11, False) * np.float32(2.0) ** np.float32(exponent)).astype(np.complex64)
    gates = [W.Gate("cp", (a, b), (0.3 + 0.1 * a + 0.01 * b,)) for a in range(5) for b in (5, 6, 9, 14, 17, 20, 21)]
    gates += CHAIN + [W.Gate("u3", (q,), (0.7 + 0.3 * q, 0.0, 0.0)) for q in qubits]
    f = P.fuse(gates, 5, coupled=True)
    assert any(len(t) == 5 and len(c[0]) > 0 for (t, _), c in zip(f.blocks(), f.couplings()))

    def run(dt, mode):
        h = P.Handle()
        h.set_tile_mode(mode)
        t = torch.from_numpy(x.astype(np.complex64 if dt == "c64" else np.complex128)).cuda()
        st = P.State(h, N, dt, basis=None, tensor=t)
        P.sv_apply_fused(st.s, f.f)
        out = st.to_numpy()
        st.close()
        h.close()
        return out

    exact = run("c128", P.SV_TILE_NARROW)
    swept, alone = (np.linalg.norm((run("c64", m) - exact) * 2.0 ** -exponent) for m in (P.SV_TILE_AUTO, P.SV_TILE_NARROW))
    f.free()
    assert 0.0 < swept <= alone, (swept, alone)
