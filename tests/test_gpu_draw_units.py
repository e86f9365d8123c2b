"""The final draw at the edges of its units: 128, 256 or 512 target ids per wavefront or several blocks of 512, one or several
workgroups per sequence, more masses than one wavefront scans at once.  Against the oracle; every case runs twice on one context, so that the
second launch finds what the first put back."""
import numpy as np
import pytest

from test_gpu_parity import _imports
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V_t,V_d,B", [
    ("f32", 2, 2, 3),               # two ids
    ("f32", 127, 40, 5),            # a ragged unit of 128
    ("f32", 2049, 500, 4),          # 17 units: two workgroups, the second with one id
    ("bf16", 65536, 3000, 2),       # 512 units of 128, the most
    ("bf16", 65537, 3000, 2),       # 257 units of 256
    ("bf16", 32000, 3001, 16),      # 250 units x 16 sequences: as many workgroups as compute units
    ("bf16", 33025, 3001, 24),      # 130 of 256, one id in the last
    ("bf16", 65600, 3001, 40),      # 129 of 512, two turns: the second of every sequence has one unit of 64 ids
    ("f32", 300000, 2000, 2),       # 1172 of 256: 19 sums of 64 masses
    ("f32", 2097153, 2000, 1),      # above 4096 units of 512: two blocks each, 2049 units
    ("f32", 4194400, 2000, 1),      # 8193 blocks of 512: three each
])
def test_units_of_the_draw(dtype, V_t, V_d, B):
    ov, ot, Verifier, parity = _imports()
    rng = np.random.default_rng(V_t)
    temps = rng.choice([1.0, 0.7], size=B).tolist()
    case = make_case(CaseSpec(name=f"units_{dtype}_{V_t}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=[1] * B, temperature=temps,
                              n_direct=int(0.8 * min(V_d, V_t)), data_seed=V_d, philox_seed=7, logits_only=True, align=0.3))
    ref = ov.verify_case(case)
    v = Verifier.for_case(case)
    try:
        for turn in range(2):
            print(f"units V_t={V_t} B={B} turn {turn}", flush=True)
            rep = parity.compare(case, v.run_case(case), ref, logits_from_gpu=False)
            assert not rep.failures, "\n".join(rep.failures[:10])
            assert rep.divergent <= 1
    finally:
        v.close()


@pytest.mark.parametrize("V_t", [2049, 40001, 300000, 4194400])
def test_empty_residual_and_the_last_id(V_t):
    """p and q' are one-hot at the same id, the first, the last of a unit or the very last: no residual mass, the draw is from p."""
    ov, ot, Verifier, parity = _imports()
    hot = [0, 127, 1024, V_t - 1]
    B, V_d = len(hot) if V_t < 10**6 else 1, 6
    hot = hot[-B:]
    case = make_case(CaseSpec(name=f"last_{V_t}", dtype="f32", d=8, V_t=V_t, V_d=V_d, k=[1] * B, temperature=[1.0] * B, n_direct=0,
                              data_seed=5, philox_seed=3, logits_only=True))
    case.direct_map[:] = -1
    case.direct_map[1:1 + B] = hot
    case.target_logits[:] = 0
    case.draft_logits[:] = 0
    case.draft_ids[:] = 0                              # no image: the proposal is empty
    for b in range(B):
        case.target_logits[2 * b, hot[b]] = 2000.0
        case.draft_logits[b, 1 + b] = 2000.0
    ref = ov.verify_case(case)
    assert ref["flags"].tolist() == [ot.OT_FLAG_UNMAPPABLE | ot.OT_FLAG_RESID_ZERO] * B
    v = Verifier.for_case(case)
    try:
        for _ in range(2):
            rep = parity.compare(case, v.run_case(case), ref, logits_from_gpu=False)
            assert not rep.failures, "\n".join(rep.failures[:10])
            assert rep.divergent == 0
    finally:
        v.close()
