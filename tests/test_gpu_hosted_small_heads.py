"""The heads that leave softmax partials of 64 columns and take the draft side in front workgroups: bf16 up to 16 rows, and fp32
with a workgroup for each piece of a draft row or, where the multiplying workgroups fill the chip, with whole rows per wavefront.
Row maxima and argmaxima are exact, sums of exponentials to 2e-6 (binary32 exponentials, each to a few 2^-24, added in binary64),
whether the launch hosts the draft side or not, and the whole step agrees with the oracle."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,V_t,V_d,ks", [
    ("bf16", 64, 65, 40, [0, 1]),                       # one tile and a ragged second; 64 of its columns are padding
    ("bf16", 1096, 1001, 1111, [5, 0, 3, 1]),           # odd rows; the hidden dimension ends inside a step
    ("bf16", 72, 33001, 40000, [14]),                   # more than 512 partials a row; draft rows of several batches
    ("bf16", 8, 4096, 24, [0] * 14 + [1]),              # a sequence per row; one step deep: most wavefronts have none
    ("f32", 33, 1024, 512, [4]),                        # a workgroup per piece
    ("f32", 20, 321, 7, [2, 0, 30, 4]),                 # draft rows shorter than their pieces
    ("f32", 17, 20011, 1003, [7, 0, 15, 9, 20]),        # whole rows by wavefronts, two row tiles
    ("f32", 16, 33003, 130, [1, 2, 0] * 30),            # more sequences than front workgroups, more than 512 partials
])
def test_partials_and_draft_side(dtype, d, V_t, V_d, ks):
    ov, ot, Verifier, parity = _imports()
    B = len(ks)
    temps, dtemps = [[1.0, 0.5, 0.0, 2.0][i % 4] for i in range(B)], [[0.8, 1.0, 1.3, 0.0][i % 4] for i in range(B)]
    case = make_case(CaseSpec(name=f"small_{dtype}_{V_t}_{B}", dtype=dtype, d=d, V_t=V_t, V_d=V_d, k=ks, temperature=temps,
                              draft_temperature=dtemps, n_direct=min(V_d, V_t) // 2, n_ngram=min(60, V_t // 8), ngram_len=(2, 4),
                              plant_cover=0.4, align=0.8, data_seed=V_t + V_d, philox_seed=4))
    ref = ov.verify_case(case)
    Zq = ov.widen(case.draft_logits, dtype).astype(np.float64)
    T = np.repeat([t or 1.0 for t in temps], np.asarray(ks) + 1)[:, None]
    Td = np.repeat([t or 1.0 for t in dtemps], ks)[:, None]
    for side in (ot.OT_DRAFT_SIDE_IN_LM_HEAD, ot.OT_DRAFT_SIDE_SEPARATE, ot.OT_DRAFT_SIDE_AUTO):
        _say(f"small head {dtype} M={case.M} d={d} V_t={V_t} V_d={V_d} draft_side={side}")
        v = Verifier.for_case(case, draft_side=side)
        try:
            structure = ot.ot_verify_structure(v.ctx, case.B, case.M)[0]
            if side != ot.OT_DRAFT_SIDE_AUTO:
                assert structure == (ot.OT_STRUCTURE_HOSTED if side == ot.OT_DRAFT_SIDE_IN_LM_HEAD else ot.OT_STRUCTURE_SEPARATE)
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
        rep = parity.compare(case, got, ref, logits_from_gpu=True)
        assert not rep.failures, "\n".join(rep.failures[:10])
        assert rep.divergent <= max(1, case.B // 100)
