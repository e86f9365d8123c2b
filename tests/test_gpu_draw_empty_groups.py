"""The final draw where its target falls into the rounding of a running sum across entries without mass.  The two halves of a
vocabulary hold the same few masses and u is exactly 1/2, so the target is the running sum at the end of the first half, in front
of empty wavefronts of a unit or empty groups of 64 units.  A scan adds in another order for every lane, so that sum can rise by a
unit in the last place across an empty entry, which must not be taken: the token is the last id of the first half or the first of
the second.  (In a model of the scan about 8 % of such sequences have their target in that step.)"""
import numpy as np
import pytest
import torch

from test_gpu_parity import _imports
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu

HALF_SEQ_ID, HALF_SEED = 23142362, 1     # u of row 0 of step 0 is exactly 1/2


@pytest.mark.parametrize("V_t,B,group", [
    (512, 1000, 64),                # one unit of 512: a wavefront on 64 ids each
    (8 * 32768, 128, 32768),        # 512 units: eight sums of 64 masses
    (8 * 8192, 8, 8192),            # the same of units of 128, several workgroups a sequence
])
def test_target_in_front_of_an_empty_group(V_t, B, group):
    from oracle.philox import uniforms
    ov, ot, Verifier, parity = _imports()
    assert uniforms(HALF_SEED, HALF_SEQ_ID, 0, 0)[1] == 0.5
    rng = np.random.default_rng(V_t)
    turns = 1 if B > 8 else 32
    case = make_case(CaseSpec(name=f"empty_{V_t}", dtype="f32", d=8, V_t=V_t, V_d=2, k=[0] * B, temperature=[1.0] * B, n_direct=0,
                              data_seed=5, philox_seed=HALF_SEED, logits_only=True))
    case.seq_id[:] = HALF_SEQ_ID
    first = group * np.array([1, 2, 3]) + 5
    second = group * np.array([5, 6, 7]) + 9
    v = Verifier.for_case(case)
    try:
        inp = v.upload(case)
        for turn in range(turns):
            z = rng.uniform(-2.5, 0.0, size=(B, 3)).astype(np.float32)
            case.target_logits[:] = -np.inf
            case.target_logits[:, first] = z
            case.target_logits[:, second] = z[:, [0, 2, 1]]
            inp["target_logits"].copy_(torch.from_numpy(case.target_logits))
            print(f"empty groups V_t={V_t} B={B} turn {turn}", flush=True)
            v.step(inp, from_logits=True)
            got = v.results(inp)["out_tokens"]
            wrong = got[(got != first[-1]) & (got != second[0])]
            assert wrong.size == 0, (wrong.size, np.unique(wrong))
    finally:
        v.close()
