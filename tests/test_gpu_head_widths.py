"""The bf16 LM head: with one M-block at every width of its workgroups (128 to 640 columns, chosen by the vocabulary so that
256 compute units run few full rounds), at the row counts where its kernel changes, ragged ends of the vocabulary and of the
hidden dimension included, and with several M-blocks at every height and width that the plan can choose: logits against
float64, and the row statistics that its epilogue leaves."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


def _check(M, V_t):
    ov, ot, Verifier, parity = _imports()
    ks = [min(40, M - r) - 1 for r in range(0, M, 40)]
    temps = [[1.0, 0.5, 0.0, 2.0][i % 4] for i in range(len(ks))]
    case = make_case(CaseSpec(name=f"width_{M}x{V_t}", dtype="bf16", d=40, V_t=V_t, V_d=64, k=ks, temperature=temps, n_direct=32,
                              data_seed=M + V_t, philox_seed=1))
    assert case.M == M
    Z = ov.lm_head_logits(case.hidden, case.W, "bf16")
    for side in (ot.OT_DRAFT_SIDE_IN_LM_HEAD, ot.OT_DRAFT_SIDE_SEPARATE):
        _say(f"head width case M={M} V_t={V_t} draft_side={side}")
        v = Verifier.for_case(case, draft_side=side)
        try:
            v.step(v.upload(case))
            ws = v.workspace(case.M, case.K, with_logits=True)
        finally:
            v.close()
        # 40 products per logit: one rounding of 2^-24 each of sums that stay below 4 times their spread
        np.testing.assert_allclose(ws["logits"], Z, rtol=1e-5, atol=5e-6)
        got = ws["logits"].astype(np.float64)
        assert np.array_equal(ws["row_max"], ws["logits"].max(axis=1)) and np.array_equal(ws["row_argmax"], got.argmax(axis=1))
        T = np.repeat([t or 1.0 for t in temps], [k + 1 for k in ks])[:, None]
        np.testing.assert_allclose(ws["row_sumexp"], np.exp((got - got.max(axis=1, keepdims=True)) / T).sum(axis=1), rtol=2e-6)


@pytest.mark.parametrize("V_t", [32768, 32769, 66001, 98500, 131073, 152064])
@pytest.mark.parametrize("M", [17, 33, 65, 97, 128, 129, 145, 176])
def test_widths(M, V_t):
    _check(M, V_t)


# at d = 40 and 256 compute units: 4, 6, 9, 10 row tiles x 256 columns in several blocks, 12 to 18 in one, 9 to 11 x 512 columns
@pytest.mark.parametrize("M,V_t", [(177, 1500), (193, 17000), (289, 17001), (433, 17000), (177, 33001), (193, 33000), (225, 33001),
                                   (257, 33002), (330, 33001), (433, 33000), (512, 33001)])
def test_several_blocks(M, V_t):
    _check(M, V_t)


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
