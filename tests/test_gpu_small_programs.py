"""Programs of few and of many blocks on small states: whichever of launches of
their own, one tile or several tiles they take, the state has the bits of one
sweep per block (a forced tile mode)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _haar(k, rng):
    q, _ = np.linalg.qr(rng.standard_normal((1 << k, 1 << k)) + 1j * rng.standard_normal((1 << k, 1 << k)))
    return q


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 4, 7, 10, 11, 12, 13])
def test_small_programs_have_the_bits_of_single_sweeps(dt, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2308_01999_amd as P
    rng = np.random.default_rng(n)
    h = P.Handle()
    st = P.State(h, n, dt)
    x = (rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)).astype(np.complex64 if dt == "c64" else np.complex128)
    for k in list(range(1, min(n, 5) + 1)) + [0]:  # 0: blocks of one to five qubits
        for count in (1, 2, 6, 7, 20):
            ks = [min(n, k or 1 + i % 5) for i in range(count)]
            gates = [(tuple(int(q) for q in rng.choice(n, size=kk, replace=False)), _haar(kk, rng), (), None) for kk in ks]
            f = P.Fused(P.sv_fuse_gates(gates, max(ks)))
            got = []
            for mode in (P.SV_TILE_AUTO, P.SV_TILE_NARROW):
                h.set_tile_mode(mode)
                P.sv_copy_from_host(st.s, x)
                P.sv_apply_fused(st.s, f.f)
                got.append(st.to_numpy())
                P.sv_copy_from_host(st.s, x)
                g = P.sv_graph_create(st.s, f.f)
                P.sv_graph_launch(g)
                h.sync()
                got.append(st.to_numpy())
                P.sv_graph_destroy(g)
            for other in got[1:]:
                np.testing.assert_array_equal(got[0], other, err_msg=f"{dt} {n} qubits, {ks}")
            f.free()
    st.close()
    h.close()
