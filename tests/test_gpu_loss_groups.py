"""The loss launch at the edges of its split: workgroups of 256, 512 and 1024 threads, the draft row in LDS or gathered from memory
(too large, or in the order of the terms), one to 64 groups of terms per row, one or several turns of eight terms per thread, the
mapped pairs or (q' wanted) all target ids as terms, rows without a token, several calls on one context."""
import numpy as np
import pytest

from test_gpu_distill import _compare, _imports
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


def _split(M, n_terms, row_bytes, local):
    """(threads, draft row in LDS, groups per row, turns) of the launch: the rule written out again, so that a case that no longer
    reaches what it is here for is noticed."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    staged = row_bytes <= (78 << 10 if local else 150 << 10)
    threads = 256 if not staged or row_bytes <= 40 << 10 else 512 if row_bytes <= 78 << 10 else 1024
    want = -(-(1024 // threads) * n_cu // M)
    if not staged:
        want = max(want, -(-n_terms // (64 * threads)))
        if not local:
            want = max(want, min(64, 128 * row_bytes // (2 << 20)))
    turns = -(-n_terms // (min(64, -(-n_terms // (8 * threads)), want) * 8 * threads))
    return threads, staged, -(-n_terms // (turns * 8 * threads)), turns


@pytest.mark.parametrize("dtype,V_t,V_d,pairs,B,k,qprime,split", [
    ("bf16", 3000, 2101, 2048, 3, 3, False, (256, True, 1, 1)),
    ("bf16", 3000, 2103, 2049, 3, 3, False, (256, True, 2, 1)),          # a second group of one pair
    ("bf16", 5200, 5001, 4097, 300, 3, False, (256, True, 1, 3)),        # rows at every 2-byte alignment in LDS
    ("bf16", 15000, 30001, 12289, 100, 4, False, (512, True, 2, 2)),
    ("bf16", 45000, 50257, 40000, 3, 3, False, (1024, True, 5, 1)),      # 100 KB per draft row
    ("f32", 30011, 32003, 24577, 90, 3, False, (1024, True, 1, 4)),      # 128 KB
    ("bf16", 6000, 76784, 3000, 3, 3, False, (1024, True, 1, 1)),        # the largest row that is copied
    ("bf16", 6000, 76785, 3000, 3, 3, False, (256, False, 2, 1)),        # one id more: gathered from memory
    ("bf16", 40000, 78000, 30000, 300, 1, False, (256, False, 8, 2)),
    ("f32", 20011, 20011, 20011, 3, 3, False, (256, False, 10, 1)),      # one vocabulary: read in the order of the terms
    ("f32", 20011, 20011, 20011, 300, 1, False, (256, False, 3, 4)),
    ("f32", 131072, 1001, 800, 2, 1, True, (256, True, 64, 1)),
    ("f32", 140001, 1001, 800, 2, 1, True, (256, True, 35, 2)),
    ("bf16", 30011, 2003, 1602, 100, 3, True, (256, True, 3, 5)),
    ("f32", 700, 5, 4, 600, 2, False, (256, True, 1, 1)),                # more rows than the chip holds workgroups
])
def test_groups_and_turns(dtype, V_t, V_d, pairs, B, k, qprime, split):
    rng = np.random.default_rng(V_t)
    temps = rng.choice([1.0, 0.7, 0.0], size=B, p=[0.5, 0.4, 0.1])
    temps[0] = 1.0
    ks = rng.integers(max(0, k - 1), k + 1, size=B)
    ks[0] = k
    one = V_t == V_d
    case = make_case(CaseSpec(name=f"groups_{dtype}_{V_t}_{V_d}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=ks.tolist(), temperature=temps.tolist(),
                              n_direct=pairs, identity_map=one, permute_frac=0.02 if one else 0.0, n_ngram=0 if one else min(200, V_d * V_d // 2),
                              ngram_len=(2, 3), plant_cover=0.0 if one else 0.3, align=0.5, data_seed=V_d, philox_seed=5, logits_only=True))
    assert _split(case.M, V_t if qprime else pairs, V_d * (2 if dtype == "bf16" else 4) + 32, one) == split
    # tolerance as in test_loss_from_logits_all_modes; totals add up to a few hundred rows
    _compare(case, rtol=2e-6, atol=1e-6, with_qprime=qprime, modes=[("fixed", "nll", False), ("target_prob", "approx_kl", False)])


def test_repeated_calls_are_identical_and_an_empty_batch_has_no_loss():
    od, ov, ot, Verifier = _imports()
    case = make_case(CaseSpec(name="groups_repeat", dtype="bf16", d=8, V_t=40000, V_d=30000, k=[5] * 8, temperature=[1.0] * 8, n_direct=25000,
                              n_ngram=100, ngram_len=(2, 3), plant_cover=0.3, data_seed=3, philox_seed=5, logits_only=True))
    assert _split(case.M, 25000, 60032, False) == (512, True, 7, 1)
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
