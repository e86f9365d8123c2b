"""The softmax statistics launch on rows that start at any element: every alignment of a 16-byte vector, chunks of 8192 that
end inside, at and just past the shift, for target rows (fp32) and draft rows (bf16 and fp32); and a step of more sequences
than the LM-head launch stages."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _run_and_compare, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V_t,V_d", [(8191, 8191), (8192, 8193), (8193, 8190), (8195, 8185), (16383, 16385), (257, 3), (5, 1), (16386, 24571)])
def test_statistics_at_every_alignment(dtype, V_t, V_d):
    ov, ot, Verifier, parity = _imports()
    ks = [7, 3, 0, 9, 2]
    temps = [1.0, 0.5, 0.0, 2.0, 0.7]
    case = make_case(CaseSpec(name=f"align_{dtype}_{V_t}_{V_d}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=ks, temperature=temps,
                              n_direct=min(V_d, V_t) // 2, data_seed=V_t + V_d, philox_seed=3, logits_only=True))
    rng = np.random.default_rng(V_t)
    Z = case.target_logits
    for r in range(case.M):                              # maxima at the ends of the row and of the chunks
        Z[r, [0, V_t - 1, min(8191, V_t - 1), min(8192, V_t - 1)][r % 4]] = 30.0 + rng.random()
    _say(f"alignment case {case.name}")
    v = Verifier.for_case(case)
    try:
        v.step(v.upload(case), from_logits=True)
        ws = v.workspace(case.M, case.K)
    finally:
        v.close()
    Zq = ov.widen(case.draft_logits, dtype)
    for what, X, shift in (("", Z.astype(np.float64), 0), ("draft_", Zq, 1)):
        T = np.repeat([t or 1.0 for t in temps], [k + 1 - shift for k in ks])[:, None]
        assert np.array_equal(ws[what + "row_max"].astype(np.float64), X.max(axis=1))
        assert np.array_equal(ws[what + "row_argmax"], X.argmax(axis=1))
        np.testing.assert_allclose(ws[what + "row_sumexp"], np.exp((X - X.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=2e-6)


@pytest.mark.parametrize("B", [255, 256, 257, 700])
def test_many_sequences(B):
    rng = np.random.default_rng(B)
    _run_and_compare(make_case(CaseSpec(name=f"many_{B}", dtype="bf16", d=8, V_t=2503, V_d=901, k=rng.integers(0, 5, size=B).tolist(),
                                        temperature=rng.choice([1.0, 0.0, 0.7], size=B).tolist(), n_direct=700, n_ngram=200, ngram_len=(2, 4),
                                        plant_cover=0.4, align=0.6, data_seed=B, philox_seed=8, logits_only=True)))


@pytest.mark.parametrize("V_d", [40000, 100001])
def test_sum_of_a_draft_row_whose_maximum_rises_from_chunk_to_chunk(V_d):
    """One finite logit in every fourth chunk of 8192, each larger than the one before: a chunk's sum is exactly 1, and what is
    left is how a sum is carried over to a larger maximum.  That factor is formed in binary64 (a few 1e-16; in binary32 it was
    off by 1e-8, once for every group of four chunks that raised the maximum)."""
    ov, ot, Verifier, parity = _imports()
    ks, temps = [7, 7, 7], [1.0, 0.7, 1.3]
    case = make_case(CaseSpec(name=f"rising_{V_d}", dtype="f32", d=8, V_t=300, V_d=V_d, k=ks, temperature=temps, n_direct=100,
                              data_seed=V_d, philox_seed=3, logits_only=True))
    rng = np.random.default_rng(V_d)
    at = np.arange(0, V_d, 4 * 8192)
    case.draft_logits[:] = -np.inf
    case.draft_logits[:, at + 5] = np.cumsum(rng.uniform(0.1, 1.0, size=(case.K, at.size)), axis=1, dtype=np.float32)
    case.draft_ids[:] = at[0] + 5
    _say(f"rising maxima case {case.name}")
    v = Verifier.for_case(case)
    try:
        v.step(v.upload(case), from_logits=True)
        ws = v.workspace(case.M, case.K)
    finally:
        v.close()
    X, T = case.draft_logits.astype(np.float64), np.repeat(case.temperature.astype(np.float64), ks)[:, None]
    np.testing.assert_allclose(ws["draft_row_sumexp"], np.exp((X - X.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=1e-13)


@pytest.mark.parametrize("B", [2, 21])                   # the multiplying workgroups take pieces; front workgroups take rows
@pytest.mark.parametrize("V_d", [1, 5, 7, 8, 9, 15, 16, 23, 601, 4093, 4096, 8001, 31999])
def test_draft_rows_of_the_lm_head_launch_at_every_alignment(B, V_d):
    """Draft rows whose statistics the LM-head launch forms: rows at every 2-byte alignment of a 16-byte vector, half of the logits
    masked (-inf), masked runs at the row's ends, the maximum at the first element, at the last, or twice."""
    ov, ot, Verifier, parity = _imports()
    ks = [9, 8] + [9] * (B - 2)
    temps = [[1.0, 0.5, 0.0, 2.0, 0.7][i % 5] for i in range(B)]
    case = make_case(CaseSpec(name=f"hosted_{B}_{V_d}", dtype="bf16", d=16, V_t=1500, V_d=V_d, k=ks, temperature=temps, n_direct=min(V_d, 1400) // 2,
                              data_seed=V_d, philox_seed=3))
    rng = np.random.default_rng(V_d)
    masked, one, big = 0xFF80, 0x3F80, 0x4120             # -inf, 1, 10
    for q, x in enumerate(case.draft_logits):
        x[rng.choice(V_d, V_d // 2, replace=False)] = masked
        if q % 7 == 0: x[:V_d // 3] = masked
        if q % 7 == 1: x[V_d // 2:] = masked
        if q % 7 == 2: x[0] = big
        if q % 7 == 3: x[-1] = big
        if q % 7 == 4: x[rng.integers(0, V_d, 2)] = big
        if q % 7 == 5: x[[0, -1]] = big
        if (x == masked).all(): x[rng.integers(0, V_d)] = one
    _say(f"hosted draft rows case {case.name}")
    v = Verifier.for_case(case, draft_side=ot.OT_DRAFT_SIDE_IN_LM_HEAD)
    try:
        v.step(v.upload(case))
        ws = v.workspace(case.M, case.K)
    finally:
        v.close()
    X = ov.widen(case.draft_logits, "bf16")
    T = np.repeat([t or 1.0 for t in temps], ks)[:, None]
    assert np.array_equal(ws["draft_row_max"].astype(np.float64), X.max(axis=1))
    assert np.array_equal(ws["draft_row_argmax"], X.argmax(axis=1))
    np.testing.assert_allclose(ws["draft_row_sumexp"], np.exp((X - X.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=2e-6)
