"""Where the fp32 head takes the draft side and where that runs behind it, at shapes whose two structures were measured well apart
(us per step, hosted / separate)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _imports

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,V_t,V_d,B,M,hosted", [
    (256, 1024, 512, 1, 5, True),            # 14.0 / 18.5: a workgroup per piece of a draft row
    (1024, 32000, 8000, 16, 64, True),       # 54.9 / 58.3
    (64, 32000, 1000, 16, 64, True),         # 19.0 / 24.8
    (1024, 100000, 32000, 1, 5, False),      # 123 / 91: a draft row outlasts the head
    (1024, 100000, 32000, 8, 32, False),     # 139 / 113
    (256, 152064, 32000, 16, 64, False),     # 97 / 81
    (64, 32000, 32000, 16, 64, False),       # 57 / 26
])
def test_fp32_takes_the_draft_side_where_that_is_faster(d, V_t, V_d, B, M, hosted):
    ov, ot, Verifier, parity = _imports()
    v = Verifier(d=d, V_t=V_t, V_d=V_d, dtype="f32", W=torch.zeros(d, V_t, device="cuda:0"),
                 direct_map=np.full(V_d, -1, np.int32), max_batch=B, max_k=15)
    try:
        assert ot.ot_verify_structure(v.ctx, B, M)[0] == (ot.OT_STRUCTURE_HOSTED if hosted else ot.OT_STRUCTURE_SEPARATE)
    finally:
        v.close()
