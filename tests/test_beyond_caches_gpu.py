"""Passes over states larger than the last-level cache (512 MiB: 26 qubits
complex64, 25 complex128) against the oracle: there the kernels move the state
past the caches, in whole cache lines, and pick by the targets' positions
which accesses that takes. Smaller states take the same kernels' cached
forms, which test_gpu_parity covers.

Tolerances as in test_gpu_parity: twice the rounding bound of one k-qubit
product (2^(k+1) real terms per amplitude) times the largest amplitude; a
diagonal layer counts as one product per phase; moved amplitudes are equal.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1704_01127_amd import qsim
from supremacy_inputs import haar_unitary, random_state

pytestmark = pytest.mark.gpu

N = {"c64": 26, "c128": 25}
U = {"c64": 2.0 ** -24, "c128": 2.0 ** -53}


@pytest.fixture(scope="module")
def states():
    """One random state per type, exactly representable in it."""
    made = {}

    def get(dt):
        if dt not in made:
            made.clear()
            psi = random_state(N[dt], 5)
            made[dt] = psi.astype(np.complex64).astype(np.complex128) if dt == "c64" else psi
        return made[dt]
    yield get
    made.clear()


def device_state(psi, dt):
    t = torch.from_numpy(psi).cuda()
    return qsim.State(N[dt], dt, init="keep", amps=t.to(torch.complex64) if dt == "c64" else t)


def check(s, ref, tol):
    _, worst = s.compare(torch.from_numpy(ref).cuda())
    assert worst <= tol, (worst, tol)


# targets: low, inside a cache line, just above one, middle and top
CLUSTERS = [(1, [0]), (1, [4]), (2, [1, 24]), (3, [2, 3, 9]), (3, [10, 17, 24]), (4, [0, 5, 11, 23]),
            (4, [7, 12, 13, 20]), (5, [0, 1, 2, 3, 4]), (5, [5, 9, 16, 20, 24]), (6, [0, 1, 2, 3, 4, 5]),
            (6, [2, 4, 8, 15, 16, 24]), (6, [3, 5, 9, 10, 20, 21])]


@pytest.mark.parametrize("variant", [1, 0], ids=["staged", "direct"])
@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_clusters(dt, variant, states):
    psi = states(dt)
    scale = float(np.max(np.abs(psi)))
    old = qsim.get_option(qsim.OPT_CLUSTER_VARIANT)
    qsim.set_option(qsim.OPT_CLUSTER_VARIANT, variant)
    try:
        for k, qs in CLUSTERS:
            if dt == "c128" and variant == 0 and k in (1, 2):
                continue  # one form only
            u = haar_unitary(k, 31 * k + qs[0])
            s = device_state(psi, dt)
            s.apply_cluster(qs, u)
            ref = oracle.apply_dense(psi.copy(), qs, u)
            check(s, ref, 2 * (2 ** (k + 1) + 2) * U[dt] * math.sqrt(2 ** k) * scale)
            del s
    finally:
        qsim.set_option(qsim.OPT_CLUSTER_VARIANT, old)


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_single_gates(dt, states):
    """Every place of a bit in a 16-byte unit, a cache line and 2 KiB."""
    n = N[dt]
    psi = states(dt)
    scale = float(np.max(np.abs(psi)))
    s, ref = device_state(psi, dt), psi.copy()
    gates = [("SY", (q,)) for q in (0, 1, 2, 3, 4, n - 1)] + [("T", (q,)) for q in (0, 2, 3, 7, 8, n - 1)]
    gates += [("CZ", q) for q in ((0, 1), (2, 8), (3, n - 1), (7, 13), (n - 2, n - 1))]
    for name, qs in gates:
        s.apply_gate((name, qs))
        oracle.apply_named(ref, name, *qs)
    check(s, ref, len(gates) * 2 * 6 * U[dt] * math.sqrt(2) * scale)


@pytest.mark.parametrize("dt", ["c64", "c128"])
def test_layers(dt, states):
    n = N[dt]
    psi = states(dt)
    scale = float(np.max(np.abs(psi)))
    pairs = [(0, 1), (3, 9), (6, 7), (8, n - 1), (12, 13)]
    phases = [(0, 0.7), (6, -1.1), (7, 2.0), (n - 1, 0.4), (15, 1.3)]
    s, ref = device_state(psi, dt), psi.copy()
    s.apply_diag(pairs, phases)
    for p in pairs:
        oracle.apply_named(ref, "CZ", *p)
    for q, t in phases:
        ref.reshape(-1, 2, 2 ** q)[:, 1] *= np.exp(1j * t)
    check(s, ref, (len(phases) + 1) * 2 * 6 * U[dt] * math.sqrt(2) * scale)
    del s
    for src in ([3, 20], [0, 1, 2, n - 3, n - 2, n - 1], list(range(4, 16)), list(range(n - 12, n))):
        dst = src[len(src) // 2:] + src[:len(src) // 2]
        s = device_state(psi, dt)
        s.permute_qubits(src, dst)
        assert np.array_equal(s.to_numpy(), oracle.permute_bits(psi, src, dst))
        del s
