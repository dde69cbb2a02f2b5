"""Timed workloads of the state-vector simulator, through its public entry points.

Six kinds of work, each what a program does with the library:
  circuit   a random grid circuit from |0...0> through State.run_circuit (schedule, matrix build,
            cluster passes), then the output statistics; the gate list is kept in the library's
            layout, as a program that runs a circuit repeatedly keeps it
  per_gate  the same circuits on a complex128 state, one launch per gate (the plain method)
  dense     a program that applies its own k-qubit unitaries, one call each (k = 1..6)
  layers    a diagonal layer (CZ and phase gates) and a relabelling of bit locations
  measure   output probabilities with their statistics, and the comparison with a reference state
  batch     many small circuits in one persistent launch
Sizes are those of the tests, the tuner and the benchmark: 12 to 30 qubits, depths 10 to 40, batches
of 14- to 24-qubit circuits.
"""
import math

import numpy as np
import torch

from paper_1704_01127_amd import qsim

S = math.sqrt(0.5)
GATE_1Q = {
    "H": ((S, S), (S, -S)),
    "SX": ((0.5 + 0.5j, 0.5 - 0.5j), (0.5 - 0.5j, 0.5 + 0.5j)),
    "SY": ((0.5 + 0.5j, -0.5 - 0.5j), (0.5 + 0.5j, 0.5 + 0.5j)),
}
T_PHASE = complex(S, S)


def listed():
    return [
        # one small circuit: the host path and the launches are what it waits for
        {"name": "circuit_12q", "kind": "circuit", "dtype": "c64", "rows": 3, "cols": 4, "depth": 16,
         "scheduler": "greedy", "kmax": 5},
        # a state that fits the caches (8 MiB)
        {"name": "circuit_20q", "kind": "circuit", "dtype": "c64", "rows": 4, "cols": 5, "depth": 25,
         "scheduler": "greedy", "kmax": 6},
        # the size at which a state leaves the last-level cache (256 MiB), odd grid
        {"name": "circuit_25q", "kind": "circuit", "dtype": "c64", "rows": 5, "cols": 5, "depth": 25,
         "scheduler": "greedy", "kmax": 6},
        # the benchmark's circuit, 8 GiB, in its form
        {"name": "circuit_30q", "kind": "circuit", "dtype": "c64", "rows": 5, "cols": 6, "depth": 25,
         "scheduler": "learned", "kmax": 7},
        # double precision, fused (4 GiB)
        {"name": "circuit_28q_c128", "kind": "circuit", "dtype": "c128", "rows": 4, "cols": 7, "depth": 25,
         "scheduler": "greedy", "kmax": 5},
        # double precision, the plain method (512 MiB)
        {"name": "per_gate_25q_c128", "kind": "per_gate", "dtype": "c128", "rows": 5, "cols": 5, "depth": 25},
        # a program's own unitaries on a small state: latency of a call
        {"name": "dense_14q", "kind": "dense", "dtype": "c64", "n": 14},
        # the same on a large one
        {"name": "dense_28q", "kind": "dense", "dtype": "c64", "n": 28},
        {"name": "dense_27q_c128", "kind": "dense", "dtype": "c128", "n": 27},
        # a layer of two-qubit phases and the local part of a qubit swap
        {"name": "layers_28q", "kind": "layers", "dtype": "c64", "n": 28, "pairs": 14, "phases": 10, "moved": 6},
        # reading a state out
        {"name": "measure_27q", "kind": "measure", "dtype": "c64", "n": 27},
        # many small circuits at once
        {"name": "batch_64", "kind": "batch", "dtype": "c64", "circuits": 64, "n_lo": 14, "n_hi": 24,
         "depth_lo": 10, "depth_hi": 40},
    ]


def draw(rng):
    kind = rng.choice(["circuit", "circuit", "circuit", "per_gate", "dense", "dense", "layers", "measure", "batch"])
    if kind in ("circuit", "per_gate"):
        c128 = kind == "per_gate" or rng.random() < 0.3
        top = 25 if kind == "per_gate" else 28 if c128 else 30
        while True:
            rows, cols = rng.randint(3, 5), rng.randint(4, 10)
            if 12 <= rows * cols <= top:
                break
        depth = rng.randint(10, 40 if rows * cols < top - 1 else 25)
        case = {"kind": kind, "dtype": "c128" if c128 else "c64", "rows": rows, "cols": cols, "depth": depth}
        if kind == "circuit":
            case["kmax"] = rng.randint(4, 5) if c128 else rng.randint(5, 7)
            case["scheduler"] = rng.choice(["greedy", "learned"])
        return case
    if kind == "dense":
        dtype = rng.choice(["c64", "c64", "c128"])
        return {"kind": kind, "dtype": dtype, "n": rng.randint(12, 28 if dtype == "c64" else 27)}
    if kind == "layers":
        dtype = rng.choice(["c64", "c128"])
        n = rng.randint(14, 28 if dtype == "c64" else 27)
        return {"kind": kind, "dtype": dtype, "n": n, "pairs": rng.randint(1, 32), "phases": rng.randint(0, 32),
                "moved": rng.randint(2, 12)}
    if kind == "measure":
        dtype = rng.choice(["c64", "c128"])
        return {"kind": kind, "dtype": dtype, "n": rng.randint(14, 27)}
    lo = rng.randint(14, 20)
    return {"kind": kind, "dtype": "c64", "circuits": rng.randint(8, 64), "n_lo": lo,
            "n_hi": rng.randint(lo, min(24, lo + 6)), "depth_lo": 10, "depth_hi": rng.randint(11, 40)}


# ---------------------------------------------------------------- inputs
def grid_circuit(rows, cols, n, depth, rng):
    """H on every qubit, then depth - 1 cycles, each with one of eight matchings of the grid's edges
    as CZ gates after a random single-qubit gate (T first, never the same twice in a row) on every
    qubit that had a CZ in the cycle before and has none in this one. The last sites are left out
    when n < rows * cols."""
    order = (("H", 0, 0), ("H", 1, 1), ("V", 0, 0), ("H", 1, 0), ("V", 1, 1), ("H", 0, 1), ("V", 1, 0), ("V", 0, 1))
    gates = [("H", (q,)) for q in range(n)]
    last, before = ["H"] * n, set()
    for t in range(1, depth):
        way, a, b = order[(t - 1) % 8]
        pairs = []
        for r in range(rows):
            for c in range(cols):
                q = r * cols + c
                if way == "H" and c + 1 < cols and (c % 2, r % 2) == (a, b) and q + 1 < n:
                    pairs.append((q, q + 1))
                if way == "V" and r + 1 < rows and (r % 2, c % 2) == (a, b) and q + cols < n:
                    pairs.append((q, q + cols))
        now = {q for p in pairs for q in p}
        for q in sorted(before - now):
            rest = ["T"] if last[q] == "H" else [g for g in ("T", "SX", "SY") if g != last[q]]
            last[q] = rest[int(rng.integers(len(rest)))]
            gates.append((last[q], (q,)))
        gates += [("CZ", p) for p in pairs]
        before = now
    return gates


def grid_of(n):
    rows = int(math.isqrt(n))
    return rows, -(-n // rows)


def batch_circuits(case, seed):
    """Sizes spread evenly over the case's range; depths and gates from the seed."""
    rng = np.random.default_rng([seed, 11])
    out = []
    for i in range(case["circuits"]):
        n = case["n_lo"] + i % (case["n_hi"] + 1 - case["n_lo"])
        rows, cols = grid_of(n)
        out.append((n, grid_circuit(rows, cols, n, int(rng.integers(case["depth_lo"], case["depth_hi"] + 1)), rng)))
    return out


def circuit_of(case, seed):
    n = case["rows"] * case["cols"]
    return n, grid_circuit(case["rows"], case["cols"], n, case["depth"], np.random.default_rng([seed, 7]))


def haar(k, rng):
    d = 2 ** k
    q, r = np.linalg.qr(rng.standard_normal((d, d)) + 1j * rng.standard_normal((d, d)))
    return np.ascontiguousarray(q * (np.diag(r) / np.abs(np.diag(r))))


def dense_gates(case, seed):
    """One k-qubit unitary of each k = 1..6 on random qubits, in random order."""
    rng = np.random.default_rng([seed, 13])
    out = []
    for k in rng.permutation(np.arange(1, 7)):
        out.append(([int(q) for q in rng.choice(case["n"], int(k), replace=False)], haar(int(k), rng)))
    return out


def layer_of(case, seed):
    rng = np.random.default_rng([seed, 17])
    n = case["n"]
    pairs = [tuple(int(q) for q in rng.choice(n, 2, replace=False)) for _ in range(case["pairs"])]
    phases = [(int(rng.integers(n)), float(rng.uniform(-3, 3))) for _ in range(case["phases"])]
    src = [int(q) for q in rng.choice(n, case["moved"], replace=False)]
    return pairs, phases, src, src[1:] + src[:1]


def random_amps(n, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    real = torch.float32 if dtype == "c64" else torch.float64
    v = torch.randn(2 ** n, 2, generator=gen, device="cuda", dtype=real).mul_(math.sqrt(0.5 / 2 ** n))
    return torch.view_as_complex(v)


# ---------------------------------------------------------------- what is in hand, and one pass
def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    if kind in ("circuit", "per_gate"):
        n, gates = circuit_of(case, seed)
        return {"case": case, "state": qsim.State(n, dtype), "gates": qsim.Gates(gates)}
    if kind == "batch":
        return {"case": case, "batch": qsim.Batch(batch_circuits(case, seed))}
    st = {"case": case, "state": qsim.State(case["n"], dtype, init="keep", amps=random_amps(case["n"], dtype, seed))}
    if kind == "dense":
        st["gates"] = dense_gates(case, seed)
    elif kind == "layers":
        st["layer"] = layer_of(case, seed)
    else:
        st["ref"] = reference_amps(st["state"].amps, case, seed)
        st["p"] = torch.empty(2 ** case["n"], device="cuda", dtype=st["ref"].real.dtype)
    return st


def reference_amps(amps, case, seed):
    """A state near `amps`: what a run is compared with."""
    return random_amps(case["n"], case["dtype"], seed + 1000003).mul_(1e-3).add_(amps)


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "circuit":
        s = st["state"]
        s.run_circuit(st["gates"], kmax=case["kmax"], scheduler=case["scheduler"], fuse_diag=True,
                      skip_trailing_diag=True, skip_initial_h=True, fused_stats=True)
        return {"amps": s.amps, "stats": s.probs()}
    if kind == "per_gate":
        s = st["state"]
        s.init("zero")
        s.run_circuit(st["gates"], scheduler="per_gate")
        return {"amps": s.amps}
    if kind == "dense":
        for qubits, mat in st["gates"]:
            st["state"].apply_cluster(qubits, mat)
        return {"amps": st["state"].amps}
    if kind == "layers":
        pairs, phases, src, dst = st["layer"]
        st["state"].apply_diag(pairs, phases)
        st["state"].permute_qubits(src, dst)
        return {"amps": st["state"].amps}
    if kind == "measure":
        stats = st["state"].probs(out=st["p"])
        return {"p": st["p"], "stats": stats, "compare": st["state"].compare(st["ref"])}
    st["batch"].run()
    return {"amps": list(st["batch"].states)}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    size = 8 if case["dtype"] == "c64" else 16
    kind = case["kind"]
    if kind in ("circuit", "per_gate"):
        # the state written once; flops of the gates on the pairs they mix
        n, gates = circuit_of(case, 0)
        mixing = sum(g[0] in GATE_1Q for g in gates) - (n if kind == "circuit" else 0)
        return {"bytes": size * 2.0 ** n, "flops": 14.0 * 2 ** n * mixing}
    if kind == "batch":
        circuits = batch_circuits(case, 0)
        return {"bytes": sum(size * 2.0 ** n for n, _ in circuits),
                "flops": sum(14.0 * 2 ** n * (sum(g[0] in GATE_1Q for g in gates) - n) for n, gates in circuits)}
    amps = 2.0 ** case["n"]
    if kind == "dense":  # every call reads and writes the state
        return {"bytes": 6 * 2 * size * amps, "flops": sum(amps * (8 * 2 ** k - 2) for k in range(1, 7))}
    if kind == "layers":
        return {"bytes": 2 * 2 * size * amps, "flops": 6 * amps}
    # probabilities: state read, p written; comparison: both states read
    return {"bytes": (3 * size + size / 2) * amps, "flops": 24 * amps}


# ---------------------------------------------------------------- the same in 64 bits
def apply_1q(psi, q, m):
    v = psi.view(-1, 2, 2 ** q)
    a, b = v[:, 0].clone(), v[:, 1].clone()
    v[:, 0].mul_(m[0][0]).add_(b, alpha=m[0][1])
    v[:, 1].mul_(m[1][1]).add_(a, alpha=m[1][0])


def bits_view(psi, qubits):
    """psi with one axis of two for each of `qubits`, the rest in between; the axis of each."""
    shape, axis, left = [], {}, int(psi.numel()).bit_length() - 1
    for q in sorted(qubits, reverse=True):
        shape += [2 ** (left - q - 1), 2]
        axis[q] = len(shape) - 1
        left = q
    return psi.view(*shape, 2 ** left), axis


def flip_cz(psi, a, b):
    v, axis = bits_view(psi, (a, b))
    v.select(axis[a], 1).select(axis[b] - (axis[b] > axis[a]), 1).neg_()


def run_gates(psi, gates):
    for name, qubits in gates:
        if name == "CZ":
            flip_cz(psi, *qubits)
        elif name == "T":
            psi.view(-1, 2, 2 ** qubits[0])[:, 1].mul_(T_PHASE)
        else:
            apply_1q(psi, qubits[0], GATE_1Q[name])
    return psi


def from_uniform(n, gates):
    """The gates after the leading layer of H on every qubit."""
    psi = torch.full((2 ** n,), 2.0 ** (-n / 2), dtype=torch.complex128, device="cuda")
    return run_gates(psi, gates[n:])


def without_trailing_diagonal(gates):
    """Gates that some later gate on one of their qubits mixes, or that mix themselves."""
    kept, mixed = [], set()
    for name, qubits in reversed(gates):
        if name in GATE_1Q:
            mixed.update(qubits)
        elif not mixed.intersection(qubits):
            continue
        kept.append((name, qubits))
    return kept[::-1]


def statistics_of(psi):
    norm = p2 = ent = 0.0
    for part in psi.split(2 ** 27):
        p = part.real.square().add_(part.imag.square())
        norm += float(p.sum())
        p2 += float(p.square().sum())
        ent -= float(torch.xlogy(p, p).sum())
    return norm, p2, ent


def exact(case, seed):
    kind = case["kind"]
    if kind in ("circuit", "per_gate"):
        n, gates = circuit_of(case, seed)
        if kind == "per_gate":
            return {"amps": from_uniform(n, gates)}
        psi = from_uniform(n, without_trailing_diagonal(gates))
        return {"amps": psi, "stats": statistics_of(psi)}
    if kind == "batch":
        return {"amps": [from_uniform(n, gates) for n, gates in batch_circuits(case, seed)]}
    psi = random_amps(case["n"], case["dtype"], seed)
    if kind == "measure":
        ref = reference_amps(psi, case, seed).to(torch.complex128)
        psi = psi.to(torch.complex128)
        norm, p2, ent = statistics_of(psi)
        p = psi.abs().square_()
        dot = complex(torch.dot(ref.conj(), psi))
        fidelity = abs(dot) ** 2 / (norm * statistics_of(ref)[0])
        return {"p": p, "stats": (norm, p2, ent), "compare": (fidelity, float((psi - ref).abs().max()))}
    psi = psi.to(torch.complex128)
    if kind == "dense":
        for qubits, mat in dense_gates(case, seed):
            k = len(qubits)
            v, axis = bits_view(psi, qubits)
            rows = [axis[q] for q in reversed(qubits)]  # bit j of the matrix index is qubits[j]
            rest = [d for d in range(v.dim()) if d not in rows]
            moved = v.permute(rows + rest)
            out = (torch.from_numpy(mat).cuda() @ moved.reshape(2 ** k, -1)).view(moved.shape)
            moved.copy_(out)
        return {"amps": psi}
    pairs, phases, src, dst = layer_of(case, seed)
    for a, b in pairs:
        flip_cz(psi, a, b)
    for q, theta in phases:
        psi.view(-1, 2, 2 ** q)[:, 1].mul_(complex(math.cos(theta), math.sin(theta)))
    v, axis = bits_view(psi, src)
    order = list(range(v.dim()))
    for a, b in zip(src, dst):  # the bit at location a moves to location b
        order[axis[b]] = axis[a]
    return {"amps": v.permute(order).reshape(-1)}
