"""The fp32 LM head at the edges of its tiles: 16 rows x 64 columns x 16 hidden indices, hidden dimension split over the
wavefronts (some of them without a block), several row blocks, rows that start at any float."""
import numpy as np
import pytest

from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d,V_t", [(1, 1, 65), (2, 15, 64), (16, 17, 1001), (17, 130, 63), (32, 131, 2050), (33, 64, 517), (48, 257, 129),
                                     (64, 1024, 1000), (65, 100, 321), (96, 36, 4099), (129, 20, 200), (200, 1022, 191)])
def test_logits(M, d, V_t):
    ov, ot, Verifier, parity = _imports()
    ks = [min(50, M - r) - 1 for r in range(0, M, 50)]
    case = make_case(CaseSpec(name=f"f32_{M}x{d}x{V_t}", dtype="f32", d=d, V_t=V_t, V_d=48, k=ks, temperature=[1.0] * len(ks), n_direct=32,
                              data_seed=M * 7 + d, philox_seed=1))
    assert case.M == M
    _say(f"f32 head M={M} d={d} V_t={V_t}")
    v = Verifier.for_case(case)
    try:
        v.step(v.upload(case))
        got = v.workspace(case.M, case.K, with_logits=True)["logits"]
    finally:
        v.close()
    H, W = case.hidden.astype(np.float64), case.W.astype(np.float64)
    # d roundings of 2^-24 of partial sums that walk up to sqrt(sum (h w)^2), eight standard deviations
    bound = 8 * 2.0 ** -24 * np.sqrt(d) * np.sqrt((H * H) @ (W * W))
    assert np.all(np.abs(got - H @ W) <= bound + 1e-30)
