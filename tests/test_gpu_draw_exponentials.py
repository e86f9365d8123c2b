"""The final draw with the draft row in LDS, as stored or (three turns and more) its exponentials: workgroups that take several
turns, of 16 wavefronts and (more sequences than compute units) of 8.  Edges: the last unit of 512 ids whole, of one id, of all but one;
draft rows at every alignment, of one and of a few ids, the longest whose exponentials fit half of LDS or all of it and the next; n-gram
overrides inside the units."""
import numpy as np
import pytest

from test_gpu_parity import _run_and_compare
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


def _copy(dtype, V_t, V_d, B):
    """(wavefronts of a workgroup, what it copies of the draft row into LDS): the plan written out again, for 512 ids a unit."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    units, lds = -(-V_t // 512), 150 << 10
    masses = (-(-units // 64) * 65 + 1) // 2 * 16
    exps = masses + 4 * (V_d + 20)
    waves = 8 if B > max(n_cu, 255) and exps <= lds // 2 else 16
    turns = -(-(-(-units // max(1, n_cu * (16 // waves) // B))) // waves)
    assert turns > 1
    if turns > 2 and exps <= lds // (16 // waves):
        return waves, "exponentials"
    return waves, "stored" if masses + V_d * (2 if dtype == "bf16" else 4) + 32 <= lds else "nothing"


@pytest.mark.parametrize("dtype,V_t,V_d,B,copy", [
    ("bf16", 4608, 1, 300, (8, "stored")),               # the second turn holds one whole unit; a draft row of one id
    ("bf16", 8192, 4001, 257, (8, "stored")),            # two whole turns
    ("bf16", 8193, 4001, 257, (8, "exponentials")),      # a third one, of one id
    ("f32", 12287, 3, 520, (8, "exponentials")),         # two rounds of 8 wavefronts, the last unit of 511 ids
    ("bf16", 8704, 1, 300, (8, "exponentials")),         # a draft row of one id, whole units only
    ("bf16", 9001, 18979, 260, (8, "exponentials")),
    ("bf16", 9001, 19048, 260, (8, "exponentials")),     # exponentials that just fit half of LDS next to 65 doubles of masses
    ("bf16", 9001, 19049, 260, (16, "stored")),          # and that do not
    ("bf16", 9001, 19500, 260, (16, "stored")),
    ("bf16", 16384, 19049, 260, (16, "stored")),         # two whole turns
    ("bf16", 16385, 19049, 260, (16, "exponentials")),
    ("f32", 40000, 37500, 120, (16, "exponentials")),
    ("bf16", 30011, 37903, 130, (16, "exponentials")),   # rows at every 2-byte alignment
    ("bf16", 30011, 38248, 130, (16, "exponentials")),   # the longest row whose exponentials fit
    ("bf16", 30011, 38249, 130, (16, "stored")),         # odd rows, copied as stored
    ("bf16", 20480, 7, 200, (16, "exponentials")),       # whole units only
])
def test_exponentials_in_lds(dtype, V_t, V_d, B, copy):
    assert _copy(dtype, V_t, V_d, B) == copy
    rng = np.random.default_rng(V_t + V_d)
    temps = rng.choice([1.0, 0.7, 0.0], size=B, p=[0.5, 0.4, 0.1]).tolist()
    case = make_case(CaseSpec(name=f"exps_{dtype}_{V_t}_{V_d}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=rng.integers(0, 3, size=B).tolist(),
                              temperature=temps, n_direct=max(1, int(0.8 * min(V_d, V_t))), n_ngram=min(200, V_d * V_d // 2), ngram_len=(2, 2),
                              plant_cover=0.4, align=0.5, data_seed=V_d, philox_seed=5, logits_only=True,
                              draft_temperature=[0.0 if b % 17 == 3 else max(t, 0.5) for b, t in enumerate(temps)]))
    _run_and_compare(case)
