"""The complex64 sweeps of 22 qubits and more multiply bf16 parts of matrices and
amplitudes: their error against a complex128 run is no larger than that of the
FP32 sweeps (a forced tile mode), also for amplitudes of very different size."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("decades", [0, 20])
def test_split_sweeps_are_as_exact_as_fp32(decades):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    n = 22
    gates = W.brickwork(n, 6, 5)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.randn(1 << n, dtype=torch.complex64, device="cuda", generator=g)
    x = x * 10.0 ** (-decades * torch.rand(1 << n, device="cuda", generator=g))
    x = (x / torch.linalg.vector_norm(x)).to(torch.complex64)

    def run(dt, mode):
        h = P.Handle()
        h.set_tile_mode(mode)
        st = P.State(h, n, dt, basis=None, tensor=x.to(torch.complex64 if dt == "c64" else torch.complex128).clone())
        st.run(gates, max_fused_qubits=5)
        out = st.to_numpy()
        st.close()
        h.close()
        return out

    exact = run("c128", P.SV_TILE_AUTO)
    split, fp32 = (np.linalg.norm(run("c64", m) - exact) for m in (P.SV_TILE_AUTO, P.SV_TILE_NARROW))
    assert 0.0 < split <= fp32, (split, fp32)


@pytest.mark.parametrize("circuit", ["qft", "cxcp", "diagheavy"])
@pytest.mark.parametrize("n", [22, 25])
def test_coupled_blocks_in_sweeps(n, circuit):
    # programs of coupled fusion, whose blocks' phases depend on qubits inside
    # and outside a sweep's tiles: against the complex128 run, no further off than
    # the sweeps of single blocks (and both within 64 blocks of 32 products)
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    gates = {"qft": lambda: W.qft(n), "cxcp": lambda: W.random_cx_cp(n, 8, n),
             "diagheavy": lambda: W.diagonal_heavy(n, 120, n)}[circuit]()
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(1 << n, dtype=torch.complex64, device="cuda", generator=g)
    x = (x / torch.linalg.vector_norm(x)).to(torch.complex64)

    def run(dt, mode):
        h = P.Handle()
        h.set_tile_mode(mode)
        st = P.State(h, n, dt, basis=None, tensor=x.to(torch.complex64 if dt == "c64" else torch.complex128).clone())
        st.run(gates, max_fused_qubits=5, coupled=True)
        out = st.to_numpy()
        st.close()
        h.close()
        return out

    exact = run("c128", P.SV_TILE_NARROW)
    swept, alone = (np.linalg.norm(run("c64", m) - exact) for m in (P.SV_TILE_AUTO, P.SV_TILE_NARROW))
    assert 0.0 < swept <= 64 * 32 * 2.0 ** -24
    assert swept <= 1.1 * alone, (swept, alone)
