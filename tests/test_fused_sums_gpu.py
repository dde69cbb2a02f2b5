"""Sums taken by a run's last cluster pass (fused_stats): which runs have them,
and what the 7-qubit pass of states beyond the caches (512 MiB: 26 qubits)
stores and sums."""
import numpy as np
import pytest
import torch

import oracle
from conftest import fp32_circuit_bound
from paper_1704_01127_amd import qsim
from supremacy_inputs import Circuit, Gate, haar_unitary, random_state

pytestmark = pytest.mark.gpu


def reread(s):
    """The sums by a pass over the state."""
    return s.probs(out=torch.empty(2 ** s.n, device="cuda"))


@pytest.mark.parametrize("qs", [[0, 1, 9, 13], [2, 3, 4, 10], [0, 1, 2, 9, 13], [0, 1, 2, 3, 4], [2, 4, 8, 11, 15],
                                [0, 1, 9, 11, 13, 15], [0, 1, 2, 3, 8, 9], [0, 1, 2, 3, 4, 5], [2, 3, 4, 5, 12, 15],
                                [1, 4, 9, 10, 12, 15]], ids=str)
def test_learned_run_sums_in_its_last_cluster(qs):
    """A learned run's last cluster takes the sums wherever its targets lie, also
    where the tune table prefers the staged kernel, which has none."""
    qsim.load_tuning()
    n, k = 16, len(qs)
    s = qsim.State(n, "c64", init="uniform")
    s.run_circuit([Gate("U", tuple(qs), haar_unitary(k, k))], kmax=k, scheduler="learned", fused_stats=True,
                  record_timings=True)
    assert [r["stats"] for r in s.op_timings() if r["kind"] == "cluster"] == [True]
    fused = s.probs()
    assert fused == pytest.approx(reread(s), rel=1e-12)


# a 7-qubit pass beyond the caches is non-temporal when its second target is at bit 4 or above,
# and pairs lanes without a target on qubit 0
SETS = [[0, 4, 9, 13, 17, 21, 25], [0, 2, 7, 12, 16, 20, 24], [3, 5, 8, 11, 16, 19, 23], [1, 3, 6, 10, 15, 18, 22]]
N = 26


def block(qs, out, seed):
    """Gates of one 7-qubit cluster and of its diagonal epilogue, which reaches the qubits in `out`."""
    gates = [Gate("U", tuple(qs[:6]), haar_unitary(6, seed)), Gate("CZ", (qs[5], qs[6])), Gate("SX", (qs[6],)),
             Gate("CZ", (qs[2], qs[6])), Gate("SY", (qs[2],))]
    return gates + [Gate("CZ", (qs[1], out[0])), Gate("T", (out[1],)), Gate("CZ", (out[0], out[1]))]


@pytest.fixture(scope="module")
def psi():
    return random_state(N, 7).astype(np.complex64).astype(np.complex128)


@pytest.mark.parametrize("qs", SETS, ids=str)
def test_seven_qubit_pass_beyond_the_caches(qs, psi):
    rest = [q for q in range(N) if q not in qs]
    second = sorted(rest[2:16:2])
    circuit = block(qs, rest[-2:], 11) + block(second, qs[3:5], 12)
    s = qsim.State(N, "c64", init="keep", amps=torch.from_numpy(psi).cuda().to(torch.complex64), kmax=7)
    opts = dict(kmax=7, scheduler="greedy", fuse_diag=True, fused_stats=True)
    ref, passes = psi.copy(), 0
    for _ in range(2):  # the builder resets the passes' tile counters
        st = s.run_circuit(circuit, **opts)
        assert st["n_clusters_by_k"][7] == 2 and st["n_ops"] == 2, st
        passes += 2
        fused = s.probs()
        assert fused == pytest.approx(reread(s), rel=1e-12)
        ref = oracle.apply(ref, Circuit(N, circuit))
        _, worst = s.compare(torch.from_numpy(ref).cuda())
        assert worst <= fp32_circuit_bound(float(np.max(np.abs(ref))), passes, 7)


@pytest.mark.parametrize("qs", SETS, ids=str)
def test_sums_repeat_bit_for_bit(qs):
    s = qsim.State(N, "c64", kmax=7)
    circuit = block(qs, [q for q in range(N) if q not in qs][-2:], 13)
    seen = set()
    for _ in range(8):
        s.init("uniform")
        st = s.run_circuit(circuit, kmax=7, scheduler="greedy", fuse_diag=True, fused_stats=True)
        assert st["n_clusters_by_k"][7] == 1 and st["n_ops"] == 1, st
        seen.add(s.probs())
    assert len(seen) == 1, seen
