"""The cluster-matrix builder against the oracle: one cluster made of many
gates of every kind (more than the 64 the builder stages at a time, dense
gates first, in the middle and last), for every width and matrix layout.

Tolerance: the cluster kernel's bound on one product (test_gpu_parity), plus
the float64 error of the matrix: every gate adds at most the bound of its own
width to each entry (entries of a unitary are at most 1), on the library's and
the oracle's side, and a row of 2^k entries meets the state.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1704_01127_amd import qsim
from supremacy_inputs import Circuit, Gate, haar_unitary, random_state

pytestmark = pytest.mark.gpu

U = {"c64": 2.0 ** -24, "c128": 2.0 ** -53}


def product_bound(u, k):
    return 2 * (2 ** (k + 1) + 2) * u * math.sqrt(2 ** k)


def one_cluster(qs, n_gates, seed):
    rng = np.random.default_rng(seed)
    k = len(qs)
    gates = []
    for i in range(n_gates):
        dense = i in (0, n_gates // 2, n_gates // 2 + 1, n_gates - 1)
        name = "U" if dense else str(rng.choice(["H", "T", "SX", "SY", "X", "Y", "Z", "CZ", "TDG", "SXDG"]))
        if name == "CZ" and k < 2:
            name = "H"
        m = min(k, 6) if name == "U" and i == 0 else int(rng.integers(1, min(k, 6) + 1)) if name == "U" else \
            2 if name == "CZ" else 1
        sel = tuple(int(q) for q in rng.choice(qs, m, replace=False))
        gates.append(Gate(name, sel, haar_unitary(m, 100 * seed + i) if name == "U" else None))
    return gates


CASES = [("c64", k, 2) for k in range(1, 8)] + [("c64", 6, 0), ("c64", 6, 1)] + [("c128", k, 2) for k in range(1, 7)]


@pytest.mark.parametrize("n_gates", [5, 64, 131])
@pytest.mark.parametrize("dt,k,k6_kernel", CASES)
def test_one_cluster_of_many_gates(dt, k, k6_kernel, n_gates):
    n = 13
    qs = sorted(int(q) for q in np.random.default_rng(k).choice(n, k, replace=False))
    gates = one_cluster(qs, n_gates, 10 * k + n_gates)
    psi = random_state(n, k)
    old = qsim.get_option(qsim.OPT_K6_KERNEL)
    qsim.set_option(qsim.OPT_K6_KERNEL, k6_kernel)
    try:
        s = qsim.State(n, dt, init="keep", amps=torch.from_numpy(psi).cuda().to(
            torch.complex64 if dt == "c64" else torch.complex128))
        given = s.to_numpy().astype(np.complex128)
        st = s.run_circuit(gates, kmax=k)
        got = s.to_numpy()
    finally:
        qsim.set_option(qsim.OPT_K6_KERNEL, old)
    assert st["n_ops"] == 1 and st["n_clusters_by_k"][k] == 1, st
    ref = oracle.apply(given.copy(), Circuit(n, gates))
    scale = float(np.max(np.abs(given)))
    matrix = 2 * sum(product_bound(U["c128"], len(g.qubits)) for g in gates) * math.sqrt(2 ** k)
    assert np.max(np.abs(got - ref)) <= (product_bound(U[dt], k) + matrix) * scale
