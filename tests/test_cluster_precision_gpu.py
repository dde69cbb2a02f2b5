"""Clusters of 4 and 5 qubits on complex64 states keep float32's own precision
whatever the matrix and the state hold: qsim_apply_cluster rounds the matrix to
float and takes any matrix, so neither a scale nor a neighbouring column may
cost digits.

Tolerance on a product: each of its 2^(k+1) real terms and partial sums is
rounded once, operands too. The roundings of a dense random row are independent,
so the error's 2-norm stays below sqrt(2^(k+1)) u times the result's; tests
allow twice that."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_1704_01127_amd import qsim
from supremacy_inputs import haar_unitary, random_state

pytestmark = pytest.mark.gpu

# one and two low targets, with and without qubit 0
CASES = [(14, [1, 7, 9, 12]), (14, [0, 2, 8, 11]), (14, [1, 4, 6, 9, 12]), (14, [0, 1, 5, 8, 11])]
# states of 512 MiB, beyond the caches
LARGE = [(26, [3, 9, 14, 22]), (26, [2, 7, 9, 14, 22])]


@pytest.fixture(params=[0, 1], ids=["direct", "staged"])
def variant(request):
    old = qsim.get_option(qsim.OPT_CLUSTER_VARIANT)
    qsim.set_option(qsim.OPT_CLUSTER_VARIANT, request.param)
    yield request.param
    qsim.set_option(qsim.OPT_CLUSTER_VARIANT, old)


def apply(n, psi, qs, mat):
    s = qsim.State(n, "c64", init="keep", amps=torch.from_numpy(psi).cuda())
    s.apply_cluster(qs, mat)
    return s.to_numpy()


def state32(n, seed):
    return random_state(n, seed).astype(np.complex64)


def bound(k):
    return 2 * math.sqrt(2 ** (k + 1)) * 2.0 ** -24


@pytest.mark.parametrize("n,qs", CASES + LARGE)
def test_permutation_moves_exactly(n, qs, variant):
    k = len(qs)
    perm = np.random.default_rng(k).permutation(2 ** k)
    mat = np.zeros((2 ** k, 2 ** k), complex)
    mat[perm, np.arange(2 ** k)] = 1
    psi = state32(n, 3)
    ref = oracle.apply_dense(psi.astype(np.complex128), qs, mat).astype(np.complex64)
    assert np.array_equal(apply(n, psi, qs, mat), ref)


@pytest.mark.parametrize("n,qs,scale", [(*c, x) for c in CASES for x in (1e-6, 1e-3, 1.0, 5e4, 1e12)] +
                         [(*c, 1e-6) for c in LARGE])
def test_matrix_of_any_scale(n, qs, scale, variant):
    k = len(qs)
    mat = scale * haar_unitary(k, 40 + k)
    psi = state32(n, 4)
    ref = oracle.apply_dense(psi.astype(np.complex128), qs, mat)
    got = apply(n, psi, qs, mat).astype(np.complex128)
    assert np.linalg.norm(got - ref) <= bound(k) * np.linalg.norm(ref)


@pytest.mark.parametrize("scale", [1e6, 1e-12, 1e-30, 0.0])
@pytest.mark.parametrize("n,qs", CASES)
def test_columns_of_any_scale(n, qs, scale, variant):
    """Columns that differ in a qubit outside the cluster, one rescaled: each keeps its own precision."""
    k = len(qs)
    mat = haar_unitary(k, 50 + k)
    full = state32(n, 5)
    for b in [q for q in range(n) if q not in qs][5:8]:
        psi = full.reshape(-1, 2, 2 ** b).copy()
        psi[:, 1] *= np.float32(scale)
        ref = oracle.apply_dense(psi.reshape(-1).astype(np.complex128), qs, mat).reshape(psi.shape)
        got = apply(n, psi.reshape(-1), qs, mat).astype(np.complex128).reshape(psi.shape)
        for side in (0, 1):
            assert np.linalg.norm(got[:, side] - ref[:, side]) <= bound(k) * np.linalg.norm(ref[:, side]), (b, side)


@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("n,qs", CASES)
def test_an_infinity_stays_in_its_column(n, qs, value, variant):
    k = len(qs)
    mat = haar_unitary(k, 60 + k)
    psi = state32(n, 6)
    want = apply(n, psi, qs, mat)
    at = 0x2b5a5a5 & (2 ** n - 1)
    psi[at] = value
    got = apply(n, psi, qs, mat)
    tmask = sum(1 << q for q in qs)
    others = (np.arange(2 ** n) & ~tmask) != (at & ~tmask)
    assert np.array_equal(got[others], want[others])
    assert not np.isfinite(got[~others]).all()
