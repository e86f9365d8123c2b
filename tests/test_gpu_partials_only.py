"""Steps of several M-blocks whose LM-head launch leaves the target rows' partials while a statistics launch takes the draft rows
and the lookups: few draft rows and many, rows off the 16-byte boundary, up to four chunks of 8192 draft logits and more, the
acceptance test in the launch of the draw and in one of its own.  Row maxima and argmaxima are exact, sums of exponentials to 2e-6 (binary32 exponentials,
each to a few 2^-24, added in binary64); the whole step against the oracle."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,V_t,V_d,ks,launches", [
    (64, 40001, 12001, [7, 8, 9] * 20, 3),              # 540 rows, two chunks a draft row; odd rows
    (64, 40001, 24577, [0, 3, 1, 3] * 60, 3),           # 660 rows, four chunks
    (64, 50001, 33001, [10] * 64, 3),                   # five chunks
    (16, 50001, 24001, [1, 2] * 127 + [40], 3),         # 255 sequences, the most
    (16, 100001, 8001, [61] * 9, 4),                    # test and draw in launches of their own
])
def test_partials_from_the_head_draft_side_behind_it(d, V_t, V_d, ks, launches):
    ov, ot, Verifier, parity = _imports()
    B = len(ks)
    temps, dtemps = [[1.0, 0.5, 0.0, 2.0][i % 4] for i in range(B)], [[0.8, 1.0, 1.3, 0.0][i % 4] for i in range(B)]
    case = make_case(CaseSpec(name=f"partials_{V_t}_{B}", dtype="bf16", d=d, V_t=V_t, V_d=V_d, k=ks, temperature=temps,
                              draft_temperature=dtemps, n_direct=min(V_d, V_t) // 2, n_ngram=100, ngram_len=(2, 4),
                              plant_cover=0.4, align=0.8, data_seed=V_t + V_d, philox_seed=4))
    assert case.M > 176
    Zq = ov.widen(case.draft_logits, "bf16").astype(np.float64)
    T = np.repeat([t or 1.0 for t in temps], np.asarray(ks) + 1)[:, None]
    Td = np.repeat([t or 1.0 for t in dtemps], ks)[:, None]
    _say(f"partials only M={case.M} d={d} V_t={V_t} V_d={V_d}")
    v = Verifier.for_case(case)
    try:
        assert ot.ot_verify_structure(v.ctx, case.B, case.M) == (ot.OT_STRUCTURE_PARTIALS, launches)
        got = v.run_case(case)
        ws = v.workspace(case.M, case.K, with_logits=True)
    finally:
        v.close()
    z = ws["logits"].astype(np.float64)
    assert np.array_equal(ws["row_max"], ws["logits"].max(axis=1)) and np.array_equal(ws["row_argmax"], z.argmax(axis=1))
    np.testing.assert_allclose(ws["row_sumexp"], np.exp((z - z.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=2e-6)
    assert np.array_equal(ws["draft_row_max"].astype(np.float64), Zq.max(axis=1))
    assert np.array_equal(ws["draft_row_argmax"], Zq.argmax(axis=1))
    np.testing.assert_allclose(ws["draft_row_sumexp"], np.exp((Zq - Zq.max(axis=1, keepdims=True)) / Td).sum(axis=1), rtol=2e-6)
    rep = parity.compare(case, got, ov.verify_case(case), logits_from_gpu=True)
    assert not rep.failures, "\n".join(rep.failures[:10])
    assert rep.divergent <= max(1, B // 100)
