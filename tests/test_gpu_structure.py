"""What the LM-head launch takes, at shapes whose structures were measured well apart (us per step)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _imports

pytestmark = pytest.mark.gpu


def _structure(dtype, d, V_t, V_d, B, M):
    ov, ot, Verifier, parity = _imports()
    v = Verifier(d=d, V_t=V_t, V_d=V_d, dtype=dtype, W=torch.zeros(d, V_t, device="cuda:0", dtype=torch.bfloat16 if dtype == "bf16"
                                                                   else torch.float32),
                 direct_map=np.full(V_d, -1, np.int32), max_batch=B, max_k=15)
    try:
        return ot.ot_verify_structure(v.ctx, B, M)[0]
    finally:
        v.close()


@pytest.mark.parametrize("d,V_t,V_d,B,M,hosted", [
    (256, 1024, 512, 1, 5, True),            # hosted 14.0, separate 18.5: a workgroup per piece of a draft row
    (1024, 32000, 8000, 16, 64, True),       # 54.9 / 58.3
    (64, 32000, 1000, 16, 64, True),         # 19.0 / 24.8
    (1024, 100000, 32000, 1, 5, False),      # 123 / 91: a draft row outlasts the head
    (1024, 100000, 32000, 8, 32, False),     # 139 / 113
    (256, 152064, 32000, 16, 64, False),     # 97 / 81
    (64, 32000, 32000, 16, 64, False),       # 57 / 26
    (64, 65536, 8000, 170, 1020, False),     # 282 / 211: seven draft rows in turn
    (64, 65536, 1000, 64, 384, True),        # 75 / 79
])
def test_fp32_head(d, V_t, V_d, B, M, hosted):
    ot = _imports()[1]
    assert _structure("f32", d, V_t, V_d, B, M) == (ot.OT_STRUCTURE_HOSTED if hosted else ot.OT_STRUCTURE_SEPARATE)


@pytest.mark.parametrize("d,V_t,V_d,B,M,structure", [
    (1024, 50000, 8000, 40, 320, "HOSTED"),          # hosted 59.7, partials alone 64.5, separate 67.7
    (4096, 20001, 8000, 24, 192, "HOSTED"),          # 51.6 / 55.6 / 56.9
    (1024, 128256, 32000, 64, 512, "PARTIALS"),      # 245 / 193 / 218
    (1024, 128256, 8000, 30, 240, "PARTIALS"),       # 129 / 114 / 116
    (1024, 100000, 32000, 80, 640, "PARTIALS"),      # 235 / 214 / 215
    (1024, 8000, 8000, 24, 192, "SEPARATE"),         # 41.7 / 28.5 / 26.0
    (4096, 8000, 8000, 30, 240, "SEPARATE"),         # 51.7 / 46.3 / 43.9
])
def test_several_m_blocks(d, V_t, V_d, B, M, structure):
    ot = _imports()[1]
    assert _structure("bf16", d, V_t, V_d, B, M) == getattr(ot, "OT_STRUCTURE_" + structure)
