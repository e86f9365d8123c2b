"""The bf16 LM head: with one M-block at every width of its workgroups (128 to 640 columns, chosen by the vocabulary so that
256 compute units run few full rounds), at the row counts where its kernel changes, ragged ends of the vocabulary and of the
hidden dimension included, and with several M-blocks at every height and width that the plan can choose: logits against
float64, and the row statistics that its epilogue leaves.  The hidden dimension is deep enough that the main loop makes
several whole trips (of 256 indices in the kernels of 128 columns and in those that take slices of 128, of 128 in the others)
and, in the former, leaves a remainder: buffers, ring and load counter are then in their steady state."""
import math
from dataclasses import replace

import numpy as np
import pytest

from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


def _case(M, V_t, d):
    ks = [min(40, M - r) - 1 for r in range(0, M, 40)]
    temps = [[1.0, 0.5, 0.0, 2.0][i % 4] for i in range(len(ks))]
    return make_case(CaseSpec(name=f"width_{M}x{V_t}", dtype="bf16", d=d, V_t=V_t, V_d=64, k=ks, temperature=temps, n_direct=32,
                              data_seed=M + V_t, philox_seed=1))


def _first_rows(case, M):
    """The same batch cut to its first M rows."""
    k = np.asarray([min(40, M - r) - 1 for r in range(0, M, 40)], np.int32)
    K = int(k.sum())
    return replace(case, B=k.size, k=k, row_off=np.concatenate([[0], np.cumsum(k + 1)]).astype(np.int32), hidden=case.hidden[:M],
                   draft_logits=case.draft_logits[:K], draft_ids=case.draft_ids[:K], temperature=case.temperature[:k.size],
                   seq_id=case.seq_id[:k.size])


def _check(case, rows):
    ov, ot, Verifier, parity = _imports()
    Z = ov.lm_head_logits(case.hidden, case.W, "bf16")
    for side in (ot.OT_DRAFT_SIDE_IN_LM_HEAD, ot.OT_DRAFT_SIDE_SEPARATE):
        v = Verifier.for_case(case, draft_side=side)
        try:
            for M in rows:
                part = _first_rows(case, M)
                _say(f"head width case M={M} V_t={case.V_t} d={case.d} draft_side={side}")
                v.step(v.upload(part))
                ws = v.workspace(M, part.K, with_logits=True)
                # d / 32 roundings of 2^-24 each of running sums that stay below 4 times their spread
                np.testing.assert_allclose(ws["logits"], Z[:M], rtol=1e-5, atol=5e-6)
                got = ws["logits"].astype(np.float64)
                assert np.array_equal(ws["row_max"], ws["logits"].max(axis=1)) and np.array_equal(ws["row_argmax"], got.argmax(axis=1))
                T = np.repeat([t or 1.0 for t in part.temperature.tolist()], part.k + 1)[:, None]
                np.testing.assert_allclose(ws["row_sumexp"], np.exp((got - got.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=2e-6)
        finally:
            v.close()


def _n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


# on 256 compute units: 128, 256, 384, 512, 640 columns (384 above 128 rows) and 640 with whole tiles
@pytest.mark.parametrize("V_t,d", [(32768, 1096), (32769, 1096), (66001, 328), (98500, 328), (131073, 328), (152064, 40)])
def test_widths(V_t, d):
    assert _n_cu() == 256
    _check(_case(176, V_t, d), [17, 33, 65, 97, 128, 129, 145, 176])


def _blocks(M, d, V_t):
    """(row tiles, columns) of the blocks that more than 176 rows run as: the plan's estimate written out again, so that a case
    that no longer reaches its kernel is noticed."""
    best = None
    for tiles, cols, outside, per_column in [(t, 256, 5.0, 1.0) for t in (4, 6, 9, 10, 12, 14, 16, 18)] + [(t, 512, 9.0, 0.83) for t in (9, 10, 11)]:
        per_cu = -(-(-(-V_t // 256) * 256) // cols)
        per_cu = -(-per_cu // 8) * 8 * -(-M // (16 * tiles)) / _n_cu()
        rounds = 0.61 + 0.39 * per_cu if per_cu < 1 else 0.42 * per_cu + 0.58 * math.ceil(per_cu)
        us = rounds * (outside + d / 3584 * (14 + 5.6 * tiles) * per_column * cols / 256)
        if best is None or us < best[0]:
            best = us, (tiles, cols)
    return best[1]


@pytest.mark.parametrize("M,V_t,d,block", [(177, 1500, 1096, (4, 256)), (385, 9000, 1096, (6, 256)), (641, 9000, 1096, (9, 256)),
                                           (577, 9000, 328, (10, 256)), (481, 17000, 328, (12, 256)), (577, 17000, 328, (14, 256)),
                                           (673, 17001, 328, (16, 256)), (513, 25000, 328, (18, 256)), (353, 33001, 328, (9, 512)),
                                           (577, 25000, 328, (10, 512)), (641, 25001, 328, (11, 512))])
def test_several_blocks(M, V_t, d, block):
    assert _blocks(M, d, V_t) == block
    _check(_case(M, V_t, d), [M])


@pytest.mark.parametrize("M,V_t", [(65, 33001), (128, 66001), (65, 131073), (257, 33002)])
def test_row_sums_of_large_logits(M, V_t):
    """The sums that the epilogue leaves, against 64-bit sums of the kernel's own logits, for rows whose maximum (about 30) times
    log2(e) / T is rounded by up to 2e-6 in binary32.  What stays are the roundings of single terms, of either sign: the
    2^x (6e-8) and its argument (2^-24 of about 8), averaged over the dozens of terms that carry a sum, and log2(e) itself (1.3e-8
    of the argument).  Measured 3.0e-8 to 3.6e-8, and 4.0e-7 to 4.7e-7 with that first rounding left in."""
    ov, ot, Verifier, parity = _imports()
    ks = [min(40, M - r) - 1 for r in range(0, M, 40)]
    case = make_case(CaseSpec(name=f"sums_{M}x{V_t}", dtype="bf16", d=40, V_t=V_t, V_d=64, k=ks, temperature=[1.0] * len(ks), n_direct=32,
                              data_seed=M + V_t, philox_seed=1, sigma_h=50.0))
    _say(f"row sums case M={M} V_t={V_t}")
    v = Verifier.for_case(case, draft_side=ot.OT_DRAFT_SIDE_IN_LM_HEAD)
    try:
        v.step(v.upload(case))
        ws = v.workspace(case.M, case.K, with_logits=True)
    finally:
        v.close()
    Z = ws["logits"].astype(np.float64)
    want = np.exp(Z - Z.max(axis=1, keepdims=True)).sum(axis=1)
    rms = np.sqrt(np.mean((ws["row_sumexp"] / want - 1.0) ** 2))
    _say(f"  rms {rms:.3g}, largest logit {Z.max():.1f}")
    assert rms < 1.2e-7
