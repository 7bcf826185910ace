"""Cases of the state-vector library's use, from the smallest calls to the largest.

A case is a dict of plain values.  Its "kind" names the path it takes through
the public entry points:

    program   a circuit fused once, then applied to |0..0> (or, for the QFT,
              to a basis state): the call a program repeats for each shot of
              a parameter study, a Trotter step or a benchmark circuit;
              "graph" replays it as a recorded graph
    circuit   a circuit given as gates, fused and applied in one call
              (State.run), as a program does with each new circuit
    request   one request of the serving workload: program, 16 Pauli strings,
              1024 samples
    batch     many small circuits in one recorded run, with their Z-type
              observables
    gates     single gates on a dense state: dense with and without controls,
              diagonal, permutation, Pauli rotation, index bit swap
    reduce    what is read from a state: Pauli strings, outcome probabilities,
              a dense observable, the norm
    sample    outcomes drawn without collapse, uniforms and outcomes on the
              device

Sizes are those of the repository's configurations, tests and benchmark
(12-, 14- and 30-qubit brickwork circuits of depth 20, 8-20 qubit batches,
10-28 qubit requests, random CNOT/CP circuits of depth 12, the QFT, 2^20
shots), with circuits that fill a smaller part of the card where a state of
the full size would only repeat the same sweep more often.
"""
import math

import numpy as np
import torch

TWO_PI = 2.0 * math.pi
COMPLEX = {"c64": torch.complex64, "c128": torch.complex128}
AMP = {"c64": 8, "c128": 16}


# ------------------------------------------------------------------ cases

def listed():
    return [
        # the smallest state of the parity configuration: launches and host work
        {"name": "program_12q_c128", "kind": "program", "circuit": "brickwork", "n": 12, "depth": 20, "dtype": "c128",
         "coupled": False, "graph": False},
        # a small program recorded once and replayed, the benchmark's replay leg
        {"name": "replay_14q_c64", "kind": "program", "circuit": "brickwork", "n": 14, "depth": 20, "dtype": "c64",
         "coupled": False, "graph": True},
        # the median request of the serving workload
        {"name": "request_16q_c64", "kind": "request", "n": 16, "depth": 40, "dtype": "c64"},
        # an ordinary circuit on random pairs whose state stays in the caches
        {"name": "program_19q_c128", "kind": "program", "circuit": "pairs", "n": 19, "depth": 25, "dtype": "c128",
         "coupled": False, "graph": False},
        # a large request: coupled fusion, odd qubit count
        {"name": "program_23q_c64_coupled", "kind": "program", "circuit": "pairs", "n": 23, "depth": 30, "dtype": "c64",
         "coupled": True, "graph": False},
        # the benchmark's headline circuit, fused and applied
        {"name": "circuit_30q_c64", "kind": "circuit", "circuit": "brickwork", "n": 30, "depth": 20, "dtype": "c64",
         "coupled": False},
        # random CNOT/CP circuit in double precision
        {"name": "circuit_28q_c128", "kind": "circuit", "circuit": "cxcp", "n": 28, "depth": 12, "dtype": "c128",
         "coupled": False},
        # the QFT with coupled fusion
        {"name": "qft_28q_c64", "kind": "program", "circuit": "qft", "n": 28, "depth": 1, "dtype": "c64",
         "coupled": True, "graph": False},
        # many independent circuits of 8-20 qubits
        {"name": "batch_512", "kind": "batch", "count": 512, "mix": 0, "n_lo": 8, "n_hi": 20, "d_lo": 10, "d_hi": 40},
        # single gates, as a program without fusion applies them
        {"name": "gates_26q_c64", "kind": "gates", "n": 26, "count": 16, "dtype": "c64"},
        # observables of a finished state
        {"name": "reduce_26q_c64", "kind": "reduce", "n": 26, "dtype": "c64", "strings": 16},
        # the benchmark's sampling step
        {"name": "sample_28q_c64", "kind": "sample", "n": 28, "dtype": "c64", "shots": 1 << 20},
    ]


def draw(rng):
    kind = rng.choice(["program", "program", "program", "circuit", "circuit", "request", "batch", "gates", "reduce",
                       "sample"])
    dtype = rng.choice(["c64", "c128"])
    if kind == "program":
        circuit = rng.choice(["brickwork", "pairs", "cxcp", "qft"])
        n = rng.randint(9, 25)
        return {"kind": kind, "circuit": circuit, "n": n, "depth": 1 if circuit == "qft" else rng.randint(6, 40),
                "dtype": dtype, "coupled": circuit == "qft" or (n >= 21 and rng.random() < 0.5),
                "graph": n <= 18 and rng.random() < 0.4}
    if kind == "circuit":
        return {"kind": kind, "circuit": rng.choice(["brickwork", "cxcp"]),
                "n": rng.randint(22, 29 if dtype == "c64" else 28), "depth": rng.randint(6, 20), "dtype": dtype,
                "coupled": False}
    if kind == "request":
        return {"kind": kind, "n": rng.randint(10, 20), "depth": rng.randint(10, 60), "dtype": "c64"}
    if kind == "batch":
        lo = rng.randint(8, 14)
        return {"kind": kind, "count": int(math.exp(rng.uniform(math.log(24), math.log(400)))),
                "mix": rng.randint(1, 999), "n_lo": lo, "n_hi": rng.randint(lo + 2, 20), "d_lo": 10, "d_hi": rng.randint(12, 40)}
    if kind == "gates":
        return {"kind": kind, "n": rng.randint(13, 27), "count": rng.randint(5, 15), "dtype": dtype}
    if kind == "reduce":
        return {"kind": kind, "n": rng.randint(11, 27), "dtype": dtype, "strings": rng.randint(3, 24)}
    return {"kind": kind, "n": rng.randint(12, 28), "dtype": dtype,
            "shots": int(math.exp(rng.uniform(math.log(500), math.log(1 << 20))))}


# --------------------------------------------------------------- circuits
#
# A gate is (name, qubits, params), qubit j being bit j of the index.

def brickwork(n, depth, rng):
    """U3 on every qubit, then CZ on neighbours, offsets alternating."""
    gates = []
    for layer in range(depth):
        ang = rng.uniform(0.0, TWO_PI, size=(n, 3))
        gates += [("u3", (q,), tuple(float(a) for a in ang[q])) for q in range(n)]
        gates += [("cz", (i, i + 1), ()) for i in range(layer % 2, n - 1, 2)]
    return gates


def pairs(n, depth, rng):
    """U3 on every qubit, then CZ or CNOT on a random matching (serving)."""
    gates = []
    for _ in range(depth):
        ang = rng.uniform(0.0, TWO_PI, size=(n, 3))
        gates += [("u3", (q,), tuple(float(a) for a in ang[q])) for q in range(n)]
        perm = [int(v) for v in rng.permutation(n)]
        gates += [("cz" if rng.random() < 0.5 else "cx", (perm[2 * j], perm[2 * j + 1]), ()) for j in range(n // 2)]
    return gates


def cxcp(n, depth, rng):
    """U3 on every qubit, then CNOT or CP(phi) on a random matching."""
    gates = []
    for _ in range(depth):
        ang = rng.uniform(0.0, TWO_PI, size=(n, 3))
        gates += [("u3", (q,), tuple(float(a) for a in ang[q])) for q in range(n)]
        perm = [int(v) for v in rng.permutation(n)]
        for j in range(n // 2):
            a, b = perm[2 * j], perm[2 * j + 1]
            gates.append(("cx", (a, b), ()) if rng.random() < 0.5 else
                         ("cp", (a, b), (float(rng.uniform(0.0, TWO_PI)),)))
    return gates


def qft(n, depth, rng):
    """H and CP ladder from the top qubit down, then the swaps."""
    gates = []
    for j in range(n - 1, -1, -1):
        gates.append(("h", (j,), ()))
        gates += [("cp", (m, j), (math.pi / float(2 ** (j - m)),)) for m in range(j - 1, -1, -1)]
    return gates + [("swap", (j, n - 1 - j), ()) for j in range(n // 2)]


CIRCUITS = {"brickwork": brickwork, "pairs": pairs, "cxcp": cxcp, "qft": qft}


def circuit_of(case, seed):
    """(gates, the basis state they start from)"""
    rng = np.random.default_rng([seed, 1])
    gates = CIRCUITS[case.get("circuit", "pairs")](case["n"], case["depth"], rng)
    return gates, int(rng.integers(0, 1 << case["n"])) if case.get("circuit") == "qft" else 0


def batch_of(case, seed):
    """(qubit counts, circuits, Z-type masks: neighbouring pairs); the sizes
    are the case's, the angles the seed's"""
    sizes, rng = np.random.default_rng(case["mix"]), np.random.default_rng([seed, 2])
    ns = [int(v) for v in sizes.integers(case["n_lo"], case["n_hi"] + 1, size=case["count"])]
    depths = [int(v) for v in sizes.integers(case["d_lo"], case["d_hi"] + 1, size=case["count"])]
    circuits = [brickwork(n, d, rng) for n, d in zip(ns, depths)]
    return ns, circuits, [[3 << q for q in range(n - 1)] for n in ns]


def pauli_strings(n, count, rng):
    """Each qubit uniform over I, X, Y, Z, redrawn when all are I."""
    terms = []
    while len(terms) < count:
        ops = rng.integers(0, 4, size=n)
        if ops.any():
            terms.append([(q, "IXYZ"[int(o)]) for q, o in enumerate(ops) if o])
    return terms


def haar(k, rng):
    d = 1 << k
    q, r = np.linalg.qr((rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d))) / math.sqrt(2.0))
    return np.ascontiguousarray(q * (np.diag(r) / np.abs(np.diag(r)))[None, :])


def gate_list(case, seed):
    """The single gates of a "gates" case, on random distinct qubits:
    (operation, qubits, controls, control values, data)."""
    rng = np.random.default_rng([seed, 3])
    n, ops = case["n"], []

    def qubits(count):
        return [int(v) for v in rng.choice(n, size=count, replace=False)]

    for k in (1, 2, 3, 4, 5, 6):
        ops.append(("dense", qubits(k), [], [], haar(k, rng)))
    for k, c in ((1, 1), (1, 2), (2, 1), (3, 1), (5, 1)):
        qs = qubits(k + c)
        ops.append(("dense", qs[:k], qs[k:], [int(v) for v in rng.integers(0, 2, size=c)], haar(k, rng)))
    for k in (2, 10):
        ops.append(("diagonal", qubits(k), [], [], np.exp(1j * rng.uniform(0, TWO_PI, 1 << k))))
    ops.append(("permutation", qubits(3), [], [], (rng.permutation(8), np.exp(1j * rng.uniform(0, TWO_PI, 8)))))
    ops.append(("rotation", [], [], [], (float(rng.uniform(0, TWO_PI)), pauli_strings(n, 1, rng)[0])))
    qs = qubits(4)
    ops.append(("swap", qs, [], [], None))
    return [ops[i] for i in rng.permutation(len(ops))[: case["count"]]]


# ---------------------------------------------------------------- prepare

_HANDLE = None


def handle():
    """The library handle of the process, on its current stream."""
    global _HANDLE
    import paper_2308_01999_amd as sv
    if _HANDLE is None:
        _HANDLE = sv.Handle()
    return _HANDLE


def dense_state(case, seed, device="cuda", dtype=None):
    """A normalised state of independent Gaussian amplitudes."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    dtype = dtype or COMPLEX[case["dtype"]]
    psi = torch.randn(1 << case["n"], dtype=dtype, device=device, generator=g)
    return psi.mul_(2.0 ** (-case["n"] / 2))


def observables(case, seed):
    rng = np.random.default_rng([seed, 4])
    n = case["n"]
    terms = pauli_strings(n, case.get("strings", 16), rng)
    if case["kind"] == "reduce":
        terms = terms + [[(q, "Z")] for q in range(n)]
    few = [int(v) for v in rng.choice(n, size=3, replace=False)]
    m = haar(3, rng)
    return terms, few, m + m.conj().T


def prepare(case, seed):
    import paper_2308_01999_amd as sv
    h = handle()
    kind = case["kind"]
    s = {"case": case, "sv": sv, "handle": h}
    if kind == "batch":
        ns, circuits, masks = batch_of(case, seed)
        # a fixed fusion width: the same program, and the same rounding, in every process
        s["batch"] = sv.Batch(h, ns, circuits, masks, max_fused_qubits=5)
        s["amps"] = sum(1 << n for n in ns)
        return s
    if kind in ("program", "circuit", "request"):
        gates, s["start"] = circuit_of(case, seed)
        st = sv.State(h, case["n"], case["dtype"])
        if kind == "circuit":
            s["gates"] = gates
        elif case.get("graph"):
            s["graph"] = sv.Graph(st, gates, 5, coupled=case["coupled"])
        else:
            s["fused"] = sv.fuse(gates, 5, coupled=case.get("coupled", False))
        s["state"] = st  # after the graph, which is to be released first
        if kind == "request":
            s["terms"] = observables(case, seed)[0]
            s["uniforms"] = np.random.default_rng([seed, 5]).random(1024)
        return s
    s["state"] = sv.State(h, case["n"], case["dtype"], basis=None, tensor=dense_state(case, seed))
    if kind == "gates":
        s["ops"] = gate_list(case, seed)
    elif kind == "reduce":
        s["terms"], s["few"], s["matrix"] = observables(case, seed)
    else:
        g = torch.Generator(device="cuda")
        g.manual_seed(seed + 7)
        s["uniforms"] = torch.rand(case["shots"], dtype=torch.float64, device="cuda", generator=g)
        s["outcomes"] = torch.empty(case["shots"], dtype=torch.int64, device="cuda")
    return s


# -------------------------------------------------------------------- run

def run(s):
    sv, case = s["sv"], s["case"]
    kind = case["kind"]
    if kind == "batch":
        values, _, _ = s["batch"].run()
        at = (s["batch"].base - s["batch"].buffer.data_ptr()) // 8
        return {"expectations": np.concatenate(values), "states": s["batch"].buffer[at: at + s["amps"]]}
    st = s["state"]
    if kind in ("program", "circuit", "request"):
        sv.sv_set_basis_state(st.s, s["start"])
        if kind == "circuit":
            st.run(s["gates"], 5, coupled=case["coupled"])
        elif "graph" in s:
            s["graph"].launch()
        else:
            sv.sv_apply_fused(st.s, s["fused"].f)
        out = {"state": st.tensor}
        if kind == "request":
            out["expectations"] = st.expect(s["terms"])
            out["samples"] = st.sample(s["uniforms"]).astype(np.int64)
        return out
    if kind == "gates":
        for what, targets, controls, values, data in s["ops"]:
            if what == "dense":
                st.apply_matrix(data, targets, controls, values)
            elif what == "diagonal":
                st.apply_gen_permutation(None, data, targets)
            elif what == "permutation":
                st.apply_gen_permutation(data[0], data[1], targets)
            elif what == "rotation":
                sv.sv_apply_pauli_rotation(st.s, data[0], data[1])
            else:
                sv.sv_swap_index_bits(st.s, [(targets[0], targets[1]), (targets[2], targets[3])])
        return {"state": st.tensor}
    if kind == "reduce":
        v = sv.sv_expect_matrix(st.s, s["matrix"], s["few"])
        return {"norm": st.norm(), "expectations": st.expect(s["terms"]),
                "probabilities": sv.sv_measure_probabilities(st.s, s["few"]),
                "parity": np.array(sv.sv_zbasis_probabilities(st.s, s["few"])), "observable": v.real}
    sv.sv_sample_device(st.s, s["uniforms"].data_ptr(), case["shots"], s["outcomes"].data_ptr())
    return {"samples": s["outcomes"]}


# ------------------------------------------------------------------- work

def gate_flops(name):
    """Real operations per amplitude of one gate."""
    return {"u3": 14.0, "h": 4.0, "cz": 0.5, "cp": 1.5, "cx": 0.0, "swap": 0.0}[name]


def work(case):
    """Programs write their state once (they start from a basis state); gates
    on a given state read and write it once; reductions read it once.  The
    operations are those of the gates as given, one by one."""
    kind = case["kind"]
    if kind == "batch":
        ns, circuits, _ = batch_of(case, 0)
        return {"bytes": float(sum(8 << n for n in ns)),
                "flops": float(sum(sum(gate_flops(g[0]) for g in c) * (1 << n) for n, c in zip(ns, circuits)))}
    dim = 1 << case["n"]
    size = float(dim * AMP[case["dtype"]])
    if kind in ("program", "circuit", "request"):
        flops = sum(gate_flops(g[0]) for g in circuit_of(case, 0)[0]) * dim
        if kind == "request":
            flops += 16 * 8.0 * dim
        return {"bytes": size, "flops": float(flops)}
    if kind == "gates":
        flops = 0.0
        for what, targets, controls, _, _ in gate_list(case, 0):
            if what == "dense":
                flops += 8.0 * (1 << len(targets)) * dim / (1 << len(controls))
            elif what != "swap":
                flops += 6.0 * dim
        return {"bytes": 2 * size, "flops": flops}
    if kind == "reduce":
        return {"bytes": size, "flops": float(dim * (8.0 * case["strings"] + case["n"] + 64 + 8))}
    return {"bytes": size + 16.0 * case["shots"], "flops": 4.0 * dim}


# ------------------------------------------------------------------ exact
#
# Plain torch in complex128.

def named_matrix(name, p):
    """(matrix on the gate's qubits, the first qubit being its lowest bit)"""
    if name == "u3":
        t, f, l = p
        c, s = math.cos(t / 2), math.sin(t / 2)
        return np.array([[c, -np.exp(1j * l) * s], [np.exp(1j * f) * s, np.exp(1j * (f + l)) * c]])
    if name == "h":
        return np.array([[1, 1], [1, -1]], dtype=np.complex128) / math.sqrt(2.0)
    if name == "cz":
        return np.diag([1, 1, 1, -1]).astype(np.complex128)
    if name == "cp":
        return np.diag([1, 1, 1, np.exp(1j * p[0])])
    if name == "cx":  # the first qubit controls
        return np.array([[1, 0, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0], [0, 1, 0, 0]], dtype=np.complex128)
    return np.array([[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]], dtype=np.complex128)


def split_dims(n, targets):
    """The state's shape with an axis of 2 for each target (top bit first),
    and the axes of `targets`."""
    shape, axes, top = [], {}, n
    for q in sorted(targets, reverse=True):
        shape += [1 << (top - q - 1), 2]
        axes[q] = len(shape) - 1
        top = q
    return shape + [1 << top], axes


def apply_exact(psi, n, m, targets):
    """m (numpy, targets[0] its lowest bit) on a complex128 state."""
    shape, axes = split_dims(n, targets)
    front = [axes[q] for q in reversed(targets)]
    rest = [a for a in range(len(shape)) if a not in front]
    d = 1 << len(targets)
    x = psi.view(shape).permute(front + rest).reshape(d, -1)
    u = torch.from_numpy(np.ascontiguousarray(m)).to(psi.device)
    y = torch.empty_like(x)
    step = 1 << 24
    for a in range(0, x.shape[1], step):
        y[:, a: a + step] = u @ x[:, a: a + step]
    back = [0] * len(shape)
    for i, a in enumerate(front + rest):
        back[a] = i
    return y.view([shape[a] for a in front + rest]).permute(back).reshape(-1)


def grow(u, at, small):
    """u (2^k x D) with `small` applied to the row bits `at`."""
    k = int(math.log2(u.shape[0]))
    shape, axes = split_dims(k, at)
    front = [axes[q] for q in reversed(at)]
    rest = [a for a in range(len(shape) + 1) if a not in front]
    full = shape + [u.shape[1]]
    x = u.reshape(full).transpose(front + rest)
    y = (small @ x.reshape(small.shape[0], -1)).reshape(x.shape)
    return y.transpose(np.argsort(front + rest)).reshape(u.shape)


def run_exact(n, gates, start, device):
    """The circuit on |start>, gates gathered on up to six qubits."""
    psi = torch.zeros(1 << n, dtype=torch.complex128, device=device)
    psi[start] = 1.0
    rest = [(set(q), q, named_matrix(name, p)) for name, q, p in gates]
    while rest:
        on, blocked, take, keep = set(), set(), [], []
        for g in rest:
            if len(blocked) < n and not (g[0] & blocked) and len(on | g[0]) <= min(6, n):
                on |= g[0]
                take.append(g)
            else:
                blocked |= g[0]
                keep.append(g)
        qs = sorted(on)
        u = np.eye(1 << len(qs), dtype=np.complex128)
        for _, q, m in take:
            u = grow(u, [qs.index(v) for v in q], m)
        psi = apply_exact(psi, n, u, qs)
        rest = keep
    return psi


def parity_sign(idx, mask):
    """(-1)^(number of bits of idx & mask) as doubles."""
    v = idx & mask
    for sh in (32, 16, 8, 4, 2, 1):
        v = v ^ (v >> sh)
    return 1.0 - 2.0 * (v & 1).double()


def pauli_masks(term):
    x = sum(1 << q for q, o in term if o in "XY")
    z = sum(1 << q for q, o in term if o in "YZ")
    return x, z, sum(1 for _, o in term if o == "Y")


def expect_exact(psi, n, terms):
    """<P> of each string, divided by the norm, in pieces of the state."""
    piece = min(1 << n, 1 << 24)
    sums, norm = [0.0] * len(terms), 0.0
    for a in range(0, 1 << n, piece):
        idx = torch.arange(a, a + piece, device=psi.device)
        left = psi[a: a + piece]
        norm += float((left.real ** 2 + left.imag ** 2).sum())
        for t, term in enumerate(terms):
            x, z, ny = pauli_masks(term)
            w = left * psi[idx ^ x].conj() if x else left * left.conj()
            w = (w.real, -w.imag, -w.real, w.imag)[ny % 4]
            sums[t] += float((w * parity_sign(idx, z)).sum())
    return np.array(sums) / norm


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "sample":
        return None
    if kind == "batch":
        ns, circuits, masks = batch_of(case, seed)
        values = []
        for n, gates in zip(ns, circuits):
            psi = run_exact(n, gates, 0, device if n > 12 else "cpu")
            p = (psi.real ** 2 + psi.imag ** 2).cpu().numpy()
            # <Z_q Z_q+1> from the marginals of neighbouring pairs
            p = p / p.sum()
            for q in range(n - 1):
                m = p.reshape(-1, 2, 2, 1 << q).sum(axis=(0, 3))
                values.append(m[0, 0] + m[1, 1] - m[0, 1] - m[1, 0])
        return {"expectations": np.array(values), "states": None}
    n = case["n"]
    if kind in ("program", "circuit", "request"):
        gates, start = circuit_of(case, seed)
        if case.get("circuit") == "qft":
            # of |x>: exp(2 pi i x y / 2^n) / 2^(n/2), the product reduced exactly
            y = torch.arange(1 << n, device=device)
            r = ((y * start) & ((1 << n) - 1)).double() * (TWO_PI / (1 << n))
            psi = torch.polar(torch.full_like(r, 2.0 ** (-n / 2)), r)
        else:
            psi = run_exact(n, gates, start, device)
        if kind == "request":
            return {"state": psi, "expectations": expect_exact(psi, n, observables(case, seed)[0]), "samples": None}
        return {"state": psi}
    psi = dense_state(case, seed, device).to(torch.complex128)
    if kind == "gates":
        for what, targets, controls, values, data in gate_list(case, seed):
            if what == "rotation":
                theta, term = data
                x, z, ny = pauli_masks(term)
                idx = torch.arange(1 << n, device=device)
                # P|j> = i^ny (-1)^(j.z) |j ^ x>
                flipped = psi[idx ^ x] * (parity_sign(idx ^ x, z) * 1.0) * (1j ** ny)
                psi = math.cos(theta) * psi + 1j * math.sin(theta) * flipped
                continue
            if what == "diagonal":
                shape, axes = split_dims(n, targets)
                rows = torch.zeros([1] * len(shape), dtype=torch.int64, device=device)
                for a, q in enumerate(targets):
                    v = [1] * len(shape)
                    v[axes[q]] = 2
                    rows = rows + (torch.arange(2, device=device) << a).view(v)
                psi = (psi.view(shape) * torch.from_numpy(data).to(device)[rows]).reshape(-1)
                continue
            if what == "permutation":
                m = np.zeros((8, 8), dtype=np.complex128)
                m[np.arange(8), data[0]] = data[1]
            elif what == "swap":
                m = np.kron(named_matrix("swap", ()), named_matrix("swap", ()))
            else:
                m, k = np.eye(1 << (len(targets) + len(controls)), dtype=np.complex128), len(targets)
                at = sum(v << i for i, v in enumerate(values)) << k
                m[at: at + (1 << k), at: at + (1 << k)] = data
            psi = apply_exact(psi, n, m, list(targets) + list(controls))
        return {"state": psi}
    terms, few, m = observables(case, seed)
    norm = float((psi.real ** 2 + psi.imag ** 2).sum())
    y = apply_exact(psi, n, m, few)
    p = psi.real ** 2 + psi.imag ** 2
    idx = torch.arange(1 << n, device=device)
    out = torch.zeros_like(idx)
    for a, q in enumerate(few):
        out |= ((idx >> q) & 1) << a
    probs = np.array([float(p[out == b].sum()) for b in range(8)])
    even = [b for b in range(8) if bin(b).count("1") % 2 == 0]
    pe = float(sum(probs[b] for b in even))
    return {"norm": norm, "expectations": expect_exact(psi, n, terms), "probabilities": probs,
            "parity": np.array([pe, float(probs.sum()) - pe]),
            "observable": float((psi.conj() * y).real.sum()) / norm}
