"""The loss launch at the edges of its split: one to sixteen groups of 8192 ids per row, one or several turns, the draft row
in LDS or (too large, or a single turn) gathered from memory, rows without a token, several calls on one context."""
import numpy as np
import pytest

from test_gpu_distill import _compare, _imports
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V_t,V_d,B", [
    ("bf16", 8192, 801, 3),          # one group, one turn
    ("bf16", 8193, 803, 3),          # a second group of one id
    ("f32", 140001, 1001, 2),        # sixteen groups at most: two turns
    ("bf16", 30011, 2003, 150),      # one group of four turns, draft rows at every 2-byte alignment in LDS
    ("bf16", 50000, 78000, 40),      # 156 KB per draft row: several turns from memory
    ("f32", 700, 5, 600),            # more rows than two workgroups per compute unit
])
def test_groups_and_turns(dtype, V_t, V_d, B):
    rng = np.random.default_rng(V_t)
    temps = rng.choice([1.0, 0.7, 0.0], size=B, p=[0.5, 0.4, 0.1]).tolist()
    case = make_case(CaseSpec(name=f"groups_{dtype}_{V_t}_{V_d}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=rng.integers(0, 4, size=B).tolist(),
                              temperature=temps, n_direct=int(0.8 * min(V_d, V_t)), n_ngram=min(200, V_d * V_d // 2), ngram_len=(2, 3),
                              plant_cover=0.3, align=0.5, data_seed=V_d, philox_seed=5, logits_only=True))
    # tolerance as in test_loss_from_logits_all_modes; totals add up to a few hundred rows
    _compare(case, rtol=2e-6, atol=1e-6, modes=[("fixed", "nll", False), ("target_prob", "approx_kl", False)])


def test_repeated_calls_are_identical_and_an_empty_batch_has_no_loss():
    od, ov, ot, Verifier = _imports()
    case = make_case(CaseSpec(name="groups_repeat", dtype="bf16", d=8, V_t=40000, V_d=900, k=[5] * 60, temperature=[1.0] * 60, n_direct=700,
                              n_ngram=100, ngram_len=(2, 3), plant_cover=0.3, data_seed=3, philox_seed=5, logits_only=True))
    v = Verifier.for_case(case)
    try:
        inp = v.upload(case)
        v.step(inp, from_logits=True)
        first = v.distill_loss(inp, from_logits=True)
        for _ in range(5):
            again = v.distill_loss(inp, from_logits=True)
            assert all(np.array_equal(first[n], again[n]) for n in first)
        none = dict(inp, B=0, M=0, row_off_host=np.zeros(1, np.int32))
        got = v.distill_loss(none, from_logits=True)
        assert (got["loss"], got["loss_dm"], got["n_dm"], got["n_ngram_tokens"]) == (0.0, 0.0, 0, 0)
    finally:
        v.close()
