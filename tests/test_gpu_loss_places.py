"""The loss launch's places: workgroups for every token of the longest window and sequence (windows of 0 and 1 token among longer ones),
row offsets as an argument up to 31 sequences; or rows one after the other (the q' rows are wanted, or windows that would leave most places
empty); rows without a token, the last of a window among them, with and without the q' rows."""
import pytest

from test_gpu_distill import _compare
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ks,qprime", [
    ([0], True), ([1], True), ([0, 0, 0], False),
    ([3, 0, 5, 1, 0, 4, 4, 2, 5], True),
    ([3, 0, 5, 1, 0, 4, 4, 2, 5], False),
    ([0], False), ([1], False),
    ([2] * 30 + [1], False),                  # the most sequences whose row offsets travel with the launch
    ([2] * 31 + [1], False),
    ([2, 0, 3] * 100, False),
    ([63] + [0] * 40, True),                  # 41 x 64 places for 104 rows: one after the other
    ([63] + [0] * 40, False),
    ([6, 0] * 4, False),                      # 48 places for 28: just places
])
def test_places(ks, qprime):
    B = len(ks)
    case = make_case(CaseSpec(name=f"places_{B}_{sum(ks)}", dtype="bf16", d=8, V_t=2300, V_d=1001, k=ks, temperature=[[1.0, 0.7, 0.0, 1.0][i % 4] if B > 1 else 1.0 for i in range(B)],
                              n_direct=800, n_ngram=100, ngram_len=(2, 3), plant_cover=0.3, align=0.5, data_seed=B + sum(ks), philox_seed=5, logits_only=True))
    _compare(case, rtol=2e-6, atol=1e-6, with_qprime=qprime, modes=[("fixed", "nll", False), ("target_prob", "approx_kl", False), ("fixed", "approx_kl", True)])
