"""The final draw of a vocabulary whose units of 1024 ids would not fit LDS: units of ten blocks of 512.  Three ids hold all of p
equally, the last of the vocabulary among them; q' is one-hot at the middle one, so the draw is between the other two, or, where
the proposal is accepted whole, among all three.  The uniforms are the oracle's."""
import numpy as np
import pytest
import torch

from test_gpu_parity import _imports

pytestmark = pytest.mark.gpu

V_T = 20_480_003


def test_draw_above_twenty_million_ids():
    from oracle.philox import uniforms
    ov, ot, Verifier, parity = _imports()
    B, seed, step = 4, 11, 3
    ids = np.array([511, 9_999_872, V_T - 1])
    k = [1, 0, 1, 0]                                        # the drafted id has no image: the residual, or a free token
    row_off = np.concatenate([[0], np.cumsum(np.asarray(k) + 1)]).astype(np.int32)
    M, K = int(row_off[-1]), sum(k)
    dm = np.full(3, -1, np.int32)
    dm[1] = ids[1]
    v = Verifier(d=1, V_t=V_T, V_d=3, dtype="f32", W=torch.zeros(1, V_T, device="cuda:0"), direct_map=dm, max_batch=B, max_k=1)
    try:
        dev = v.device
        z = torch.full((M, V_T), -float("inf"), device=dev)
        z[:, torch.from_numpy(ids).to(dev)] = 0.0
        zq = torch.zeros(K, 3, device=dev)
        zq[:, 1] = 1000.0
        inp = {"B": B, "M": M, "K": K, "step": step, "seed": seed, "row_off_host": row_off,
               "row_off": torch.from_numpy(row_off).to(dev), "hidden": None, "target_logits": z, "draft_logits": zq,
               "draft_ids": torch.zeros(K, dtype=torch.int32, device=dev), "temperature": torch.ones(B, device=dev),
               "draft_temperature": None, "seq_id": torch.arange(B, dtype=torch.int64, device=dev), "out": v.alloc_outputs(B, M)}
        for turn in range(2):                               # the second launch finds what the first put back
            print(f"vast vocabulary turn {turn}", flush=True)
            v.step(inp, from_logits=True)
            got = v.results(inp)
            for b in range(B):
                u = uniforms(seed, b, step, 0)[1]
                among = ids[[0, 2]] if k[b] else ids
                assert got["out_tokens"][row_off[b]] == among[int(u * len(among))], (turn, b, u)
                assert got["flags"][b] == (ot.OT_FLAG_UNMAPPABLE if k[b] else 0)
    finally:
        v.close()
