"""The fp32 head on bf16 thirds (more than 16 rows, 384 hidden indices or more): edges of its blocks of 32, 48 and 64 rows, of its steps of
32 hidden indices and their split over four wavefronts; operands that do not survive the split; the draft side by few front workgroups."""
import numpy as np
import pytest

import test_gpu_hosted_small_heads as hosted
from test_gpu_parity import _imports, _say
from workloads import CaseSpec, make_case

pytestmark = pytest.mark.gpu


def _row_tiles(M, V_t):
    """Row tiles of the blocks that M rows run as: the plan's estimate written out again, so that a case that no longer reaches its
    kernel is noticed."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    tiles, wtiles = -(-M // 16), -(-V_t // 64)
    return min((2, 3, 4), key=lambda mt: -(-wtiles * -(-tiles // mt) // n_cu) * (2.0 + 2.5 * mt))


def _front(M, d, V_t, B, K):
    """(draft-side jobs, front workgroups) of a hosting launch: the plan written out again.  Three jobs a draft row have a workgroup
    each, one or two are taken by the front's wavefronts."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert M > 16 and d >= 384
    tiles = _row_tiles(M, V_t)
    workgroups = -(-(-(-V_t // 64)) // 8) * 8 * -(-M // (16 * tiles))
    if workgroups + B + 3 * K <= 2 * n_cu:
        return 3 * K, B + 3 * K
    at_once = n_cu * (3 if tiles == 2 else 2)
    want = min(32, -(-max(B, -(-K // 4)) // 8) * 8)
    room = (-(-workgroups // at_once) * at_once - workgroups) // 8 * 8
    front = min(want, room) if room >= 8 else want
    return (2 * K if -(-2 * K // (4 * front)) < 2 * -(-K // (4 * front)) else K), front


def _logits(case):
    ov, ot, Verifier, parity = _imports()
    v = Verifier.for_case(case)
    try:
        v.step(v.upload(case))
        return v.workspace(case.M, case.K, with_logits=True)["logits"]
    finally:
        v.close()


def _bound(H, W):
    """d roundings of 2^-24 of partial sums that walk up to sqrt(sum (h w)^2), eight standard deviations; what is left out, at most
    2^-24 of each product."""
    return 8 * 2.0 ** -24 * np.sqrt(H.shape[1]) * np.sqrt((H * H) @ (W * W)) + 2.0 ** -24 * (np.abs(H) @ np.abs(W))


def _case(M, d, V_t):
    ks = [min(50, M - r) - 1 for r in range(0, M, 50)]
    return make_case(CaseSpec(name=f"thirds_{M}x{d}x{V_t}", dtype="f32", d=d, V_t=V_t, V_d=48, k=ks, temperature=[1.0] * len(ks), n_direct=32,
                              data_seed=M * 7 + d, philox_seed=1))


@pytest.mark.parametrize("M,d,V_t,tiles", [
    (17, 512, 65, 2), (32, 513, 129, 2), (48, 543, 16001, 3), (49, 528, 200, 2), (64, 560, 16385, 2), (80, 1023, 8001, 3),
    (129, 545, 320, 2), (260, 640, 2050, 3), (33, 385, 3001, 2), (50, 512, 8257, 4), (64, 530, 8257, 4), (40, 1023, 16001, 3),
])
def test_logits(M, d, V_t, tiles):
    assert _row_tiles(M, V_t) == tiles
    case = _case(M, d, V_t)
    # values over many binades: every third of an operand takes part
    rng = np.random.default_rng(M + d)
    case.hidden *= np.exp2(rng.integers(-12, 13, size=case.hidden.shape)).astype(np.float32)
    _say(f"thirds M={M} d={d} V_t={V_t}")
    got = _logits(case)
    H, W = case.hidden.astype(np.float64), case.W.astype(np.float64)
    assert np.all(np.abs(got - H @ W) <= _bound(H, W) + 1e-30)


@pytest.mark.parametrize("M,d,V_t,tiles", [(50, 512, 400, 2), (50, 530, 400, 2), (48, 530, 16001, 3), (50, 512, 8257, 4), (50, 530, 8257, 4)])
def test_operands_that_are_not_finite(M, d, V_t, tiles):
    assert _row_tiles(M, V_t) == tiles
    case = _case(M, d, V_t)
    case.W[:, :] = np.where(case.W == 0, 0.01, case.W)
    case.hidden[:, :] = np.where(case.hidden == 0, 0.5, case.hidden)
    case.hidden[3, 7] = np.inf                # a whole row of infinities
    case.hidden[20, d - 1] = -np.inf
    case.hidden[33, 100] = np.nan
    case.W[5, 70] = np.inf                    # a column
    case.W[6, 200] = np.nan
    case.hidden[40, 9], case.W[9, 300] = 2e38, 1e30   # a product beyond binary32
    _say(f"thirds, operands that are not finite, M={M} d={d} V_t={V_t}")
    got = _logits(case)
    with np.errstate(all="ignore"):
        H, W = case.hidden.astype(np.float64), case.W.astype(np.float64)
        want = np.empty((M, V_t))
        for v in range(V_t):
            p = H * W[:, v]
            want[:, v] = np.where(np.abs(p) > 3.4028235e38, np.sign(p) * np.inf, p).sum(axis=1)
    want[np.abs(want) > 3.4028235e38] *= np.inf
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    with np.errstate(all="ignore"):
        bound = _bound(H, W)
    assert np.all(np.abs(got[ok] - want[ok]) <= bound[ok] + 1e-30)


@pytest.mark.parametrize("M,d,V_t,tiles", [(17, 512, 321, 2), (48, 543, 16001, 3), (50, 530, 8257, 4)])
def test_single_products(M, d, V_t, tiles):
    """Hidden rows with one value each: a logit is one product.  What the six products leave out is at most 2^-24 of it, the sum is
    rounded to binary32 (at most 2^-23 of it, however), and neither leans to a side."""
    assert _row_tiles(M, V_t) == tiles
    case = _case(M, d, V_t)
    rng = np.random.default_rng(M + d)

    def values(shape):
        mantissa = rng.integers(0, 1 << 23, size=shape)
        mantissa.flat[::5] = 0x00FFFF                     # 1 + 2^-7 - 2^-23: the two lower thirds as large as they get
        mantissa.flat[1::5] = 0x7FFFFF
        x = np.ldexp(1.0 + mantissa * 2.0 ** -23, rng.integers(-12, 13, size=shape)) * rng.choice([-1, 1], size=shape)
        return x.astype(np.float32)

    case.hidden[:] = 0
    at = rng.integers(0, d, size=M)
    at[:2] = 0, d - 1
    case.hidden[np.arange(M), at] = values(M)
    case.W[:] = values((d, V_t))
    _say(f"thirds, single products M={M} d={d} V_t={V_t}")
    got = _logits(case)[:, :V_t].astype(np.float64)
    want = case.hidden[np.arange(M), at].astype(np.float64)[:, None] * case.W[at].astype(np.float64)
    off = (got / want - 1) * 2.0 ** 24
    assert np.abs(off).max() <= 3
    # Where the weight's mantissa is random: 0.7 at most each, root mean square (0.58 of a rounding at the lower end of a binade, 0.3 left
    # out), so that the mean of 3000 and more stays below 0.013 (one deviation)
    random = (np.arange(d * V_t).reshape(d, V_t)[at] % 5 > 1)
    assert random.sum() >= 3000 and abs(off[random].mean()) <= 0.1


@pytest.mark.parametrize("up_hidden", [True, False])
def test_operands_whose_lower_thirds_are_denormal(up_hidden):
    case = _case(40, 600, 300)
    up, down = (case.hidden, case.W) if up_hidden else (case.W, case.hidden)
    up *= np.float32(2.0 ** 110)
    down *= np.float32(2.0 ** -116)           # thirds of 2^-116 - 16 and less, down to denormals themselves
    _say(f"thirds, denormal parts, up_hidden={up_hidden}")
    got = _logits(case)
    H, W = case.hidden.astype(np.float64), case.W.astype(np.float64)
    assert np.all(np.abs(got - H @ W) <= _bound(H, W))


def test_small_logits():
    """Weights about 2^-116 and ordinary hidden states: the last third of a weight is rounded to a multiple of 2^-133, to either side."""
    case = _case(40, 600, 300)
    case.W *= np.float32(2.0 ** -110)
    _say("thirds, small logits")
    got = _logits(case)
    H, W = case.hidden.astype(np.float64), case.W.astype(np.float64)
    # eight standard deviations of the roundings of the last thirds, 0.29 * 2^-133 each
    last = 8 * 0.29 * 2.0 ** -133 * np.sqrt((H * H).sum(axis=1, keepdims=True))
    assert np.all(np.abs(got - H @ W) <= _bound(H, W) + last)


@pytest.mark.parametrize("V_t,V_d,ks,tiles,jobs_a_row,front", [
    (32001, 9001, [3] * 16, 4, 2, 8),         # halves of draft rows of several batches, two sequences a front workgroup
    (32001, 40, [3] * 16, 4, 2, 8),           # halves shorter than a batch
    (32001, 7, [3] * 16, 4, 2, 8),            # second halves of no elements
    (32001, 40, [0, 1, 2] * 30, 4, 1, 24),    # 90 sequences: lookups by wavefronts; whole rows shorter than a batch
    (32001, 4099, [23], 2, 1, 8),             # blocks of 32 rows, one sequence, whole rows of several batches
    (24577, 4099, [23], 2, 3, 70),            # the same by a workgroup for every third of a row
    (32001, 2100, [15] * 3, 3, 2, 8),         # blocks of 48 rows
])
def test_draft_side_of_few_front_workgroups(V_t, V_d, ks, tiles, jobs_a_row, front):
    K = sum(ks)
    assert _row_tiles(K + len(ks), V_t) == tiles
    assert _front(K + len(ks), 400, V_t, len(ks), K) == (jobs_a_row * K, front)
    hosted.test_partials_and_draft_side("f32", 400, V_t, V_d, ks)
