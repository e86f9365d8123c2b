"""The final draw when a workgroup takes several turns of eight tiles: enough sequences that the launch would otherwise
hold more workgroups than compute units.  Against the oracle, with the draft row in LDS and (a row too large) without."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _run_and_compare
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,V_t,V_d,B", [
    ("bf16", 40001, 4001, 120),      # 3 turns, 2 groups; rows at every 2-byte alignment, last tile of 65 ids
    ("f32", 40000, 4003, 120),       # rows at every 4-byte alignment
    ("bf16", 8193, 3000, 300),       # 9 tiles in one group, the second turn holds a single tile of one id
    ("bf16", 45000, 50257, 64),      # 100 KB per draft row in LDS
    ("f32", 45000, 32003, 64),       # 128 KB
    ("bf16", 70000, 76001, 64),      # 152 KB: next to the tiles' masses about the largest that is copied
    ("bf16", 70000, 78000, 64),      # 156 KB: gathered from memory
    ("f32", 30000, 5, 300),          # a draft row shorter than two 16-byte chunks
])
def test_several_turns_per_workgroup(dtype, V_t, V_d, B):
    rng = np.random.default_rng(V_t)
    temps = rng.choice([1.0, 0.7, 0.0], size=B, p=[0.5, 0.4, 0.1]).tolist()
    case = make_case(CaseSpec(name=f"turns_{dtype}_{V_t}_{V_d}", dtype=dtype, d=8, V_t=V_t, V_d=V_d, k=rng.integers(0, 4, size=B).tolist(),
                              temperature=temps, n_direct=int(0.8 * min(V_d, V_t)), n_ngram=min(200, V_d * V_d // 2), ngram_len=(2, 3),
                              plant_cover=0.3, align=0.5, data_seed=V_d, philox_seed=5, logits_only=True,
                              draft_temperature=[0.0 if b % 17 == 3 else max(t, 0.5) for b, t in enumerate(temps)]))
    _, ref, _ = _run_and_compare(case)
    drawn = np.asarray(case.temperature) > 0
    assert (ref["n_accept"][drawn] < ref["n_mapped"][drawn]).any() and (ref["n_accept"][drawn] == ref["n_mapped"][drawn]).any()


def test_empty_residual_over_several_turns():
    """Every residual underflows to zero mass: the draw is from p (9 tiles in one workgroup, the last ragged)."""
    ov, ot, Verifier, parity = _imports()
    B, V_t, V_d = 300, 8200, 40
    case = make_case(CaseSpec(name="turns_zero", dtype="f32", d=8, V_t=V_t, V_d=V_d, k=[1] * B, temperature=[1.0] * B, n_direct=0,
                              data_seed=92, philox_seed=10, logits_only=True))
    hot = (np.arange(B) * 137 + 5) % V_t               # p and q' are one-hot at a target id of each sequence's own tile
    case.direct_map[:] = -1
    spread = np.unique(hot)[:V_d - 1]
    case.direct_map[1:1 + spread.size] = spread
    case.target_logits[:] = 0
    case.draft_logits[:] = 0
    for b in range(B):
        d = 1 + b % spread.size
        case.target_logits[2 * b, case.direct_map[d]] = 2000.0
        case.draft_logits[b, d] = 2000.0
    case.draft_ids[:] = 0                              # no image: the proposal is empty
    gpu, ref, _ = _run_and_compare(case)
    assert np.all(gpu["flags"] == (ot.OT_FLAG_UNMAPPABLE | ot.OT_FLAG_RESID_ZERO))


def test_flags_of_a_sequence_drawn_by_several_workgroups():
    """The draw adds a bit to flags that another workgroup of the same launch wrote: every bit of this step arrives, whatever
    the output buffer held before.  Five workgroups per sequence; empty residuals, ordinary ones, a free token, a greedy
    sequence and one with a drafted id out of range."""
    ov, ot, Verifier, parity = _imports()
    B, V_t, V_d = 8, 40001, 40
    case = make_case(CaseSpec(name="flags_groups", dtype="f32", d=8, V_t=V_t, V_d=V_d, k=[1] * B, temperature=[1.0] * 6 + [0.0, 1.0],
                              n_direct=0, data_seed=95, philox_seed=12, logits_only=True))
    case.direct_map[:] = -1
    case.direct_map[1:7] = [3, 9000, 17001, 25003, 33004, V_t - 1]
    case.target_logits[:] = 0
    case.draft_logits[:] = 0
    case.draft_ids[:] = 0                              # no image: the proposal is empty
    for b in range(3):                                 # p and q' are one-hot at the same id
        case.target_logits[2 * b, case.direct_map[1 + 2 * b]] = 2000.0
        case.draft_logits[b, 1 + 2 * b] = 2000.0
    case.draft_ids[5] = 1                              # its image has all of p: accepted, then a free token
    case.target_logits[10, case.direct_map[1]] = 2000.0
    case.draft_ids[7] = V_d
    ref = ov.verify_case(case)
    both = ot.OT_FLAG_UNMAPPABLE | ot.OT_FLAG_RESID_ZERO
    assert ref["flags"].tolist() == [both] * 3 + [ot.OT_FLAG_UNMAPPABLE] * 2 + [0, ot.OT_FLAG_UNMAPPABLE, ot.OT_FLAG_BAD_ID]
    v = Verifier.for_case(case)
    try:
        inp = v.upload(case)
        for before in (0, -1, both, ot.OT_FLAG_BAD_ID):
            inp["out"]["flags"].fill_(before)
            v.step(inp, from_logits=True)
            got = v.results(inp)
            rep = parity.compare(case, got, ref, logits_from_gpu=False)
            assert not rep.failures and rep.exact == B, rep.failures
            assert np.array_equal(got["flags"], ref["flags"])
    finally:
        v.close()


@pytest.mark.parametrize("temperature", [0.7, 0.9, 1.0, 1.1])
def test_masked_logits(temperature):
    """Logits of -inf (a caller's mask) on both sides: those ids have no mass, the others keep theirs, whether the low part of
    log2(e) / T rounds up or down."""
    ov, ot, Verifier, parity = _imports()
    B, V_t, V_d = 40, 9001, 2003
    case = make_case(CaseSpec(name=f"masked_{temperature}", dtype="f32", d=8, V_t=V_t, V_d=V_d, k=[3] * B, temperature=[temperature] * B,
                              n_direct=1600, n_ngram=100, ngram_len=(2, 3), plant_cover=0.3, align=0.6, data_seed=21, philox_seed=5,
                              logits_only=True))
    rng = np.random.default_rng(3)
    for row, x in enumerate(case.draft_logits):
        x[np.setdiff1d(rng.choice(V_d, V_d // 2, replace=False), case.draft_ids[row])] = -np.inf
    case.target_logits[:, rng.choice(V_t, V_t // 3, replace=False)] = -np.inf
    gpu, ref, _ = _run_and_compare(case)
    drawn = ref["out_tokens"][ref["final_row"]]
    assert np.isfinite(case.target_logits[ref["final_row"], drawn]).all() and (ref["n_accept"] < ref["n_mapped"]).any()


@pytest.mark.parametrize("B", [3, 120])                  # five workgroups of one turn, two of three turns
def test_tiles_without_residual_mass(B):
    """q' above p over a whole tile and over half of another: those have no residual mass, next to tiles that do (a draw from the
    residual) and in sequences that have none anywhere (a draw from p)."""
    ov, ot, Verifier, parity = _imports()
    V_t, V_d = 40001, 1600
    case = make_case(CaseSpec(name=f"no_mass_{B}", dtype="f32", d=8, V_t=V_t, V_d=V_d, k=[1] * B, temperature=[1.0] * B, n_direct=0,
                              data_seed=96, philox_seed=14, logits_only=True))
    case.direct_map[:] = -1
    case.direct_map[1:1025] = np.arange(1024, 2048)
    case.direct_map[1025:1537] = np.arange(5 * 1024, 5 * 1024 + 512)
    case.target_logits[:] = 0
    case.draft_logits[:] = 0
    case.draft_ids[:] = 0                                # no image: the proposal is empty
    for b in range(0, B, 3):                             # half of p and half of q' each on two ids of different tiles
        case.target_logits[2 * b] = -2000.0
        case.target_logits[2 * b, case.direct_map[[7, 1030]]] = 0
        case.draft_logits[b] = -2000.0
        case.draft_logits[b, [7, 1030]] = 0
    gpu, ref, _ = _run_and_compare(case)
    both = ot.OT_FLAG_UNMAPPABLE | ot.OT_FLAG_RESID_ZERO
    assert gpu["flags"].tolist() == [both if b % 3 == 0 else ot.OT_FLAG_UNMAPPABLE for b in range(B)]
    assert B < 10 or np.unique(gpu["out_tokens"][0::6]).size == 2          # both of them are drawn
