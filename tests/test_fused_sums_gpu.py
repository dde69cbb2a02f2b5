"""Sums taken by a run's last cluster pass (fused_stats): which runs have them."""
import pytest
import torch

from paper_1704_01127_amd import qsim
from supremacy_inputs import Gate, haar_unitary

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
