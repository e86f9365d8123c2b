"""Performance cases: the calls that a program which verifies drafted tokens makes, over the range of their sizes.

Every case is a dict of plain values.  `call` says which entry point a pass goes through:

  step       Verifier.step from the target's hidden states (LM head, statistics, translation, test, final draw)
  logits     Verifier.step(from_logits=True): the caller has projected the hidden states itself
  loss       Verifier.distill_loss on a batch that a step has just verified (online training of the drafter)
  adapt      ot_adaptive_drafting: stop rule and the acceptance head's loss value for one batch
  iteration  a step, then ot_ngram_cache_insert of the n-grams that the iteration found (full cache, LRU eviction)

Inputs have the shapes and the distributions of workloads/synth.py (N(0, 1) hidden states, N(0, 0.02^2) weights,
N(0, 2^2) draft logits, drafted ids sampled from the drafter's distribution, n-gram keys with a long-tailed use), made on
the GPU from the seed; about two thirds of the proposed tokens are agreeable to the target, so that acceptance runs of
several tokens, rejections inside the window and free tokens all occur.  A step also returns the logits and the row
statistics that it leaves in the context's workspace.
"""
import math

import numpy as np
import torch

from paper_2507_02659_amd import binding as ot
from paper_2507_02659_amd.runner import Verifier

DEVICE = "cuda:0"
SIGMA_W, SIGMA_Q, ALIGN, COVER = 0.02, 2.0, 0.65, 0.30


# ------------------------------------------------------------------------------------------------ the cases
def _case(name, call, dtype, d, V_t, V_d, B, k_min, k_max, **more):
    c = {"call": call, "dtype": dtype, "d": d, "V_t": V_t, "V_d": V_d, "B": B, "k_min": k_min, "k_max": k_max,
         "temperature": 1.0, "greedy": 0.0, "entries": 0, "max_len": 2, "qprime": False, "approx_kl": False}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # one sequence of a toy fp32 model: nothing but launches and latency
        _case("step_f32_toy", "step", "f32", 256, 1024, 512, 1, 4, 4, entries=64, max_len=3),
        # one interactive sequence, drafter and target of one family (shared 32000-id vocabulary)
        _case("step_b1_v32k", "step", "bf16", 4096, 32000, 32000, 1, 5, 5),
        # the whole online iteration of one interactive sequence on a 152064-id target: step, then the cache update
        _case("iteration_b1_v152k", "iteration", "bf16", 3584, 152064, 32000, 1, 5, 5, entries=20000, max_len=4),
        # a handful of sequences with ragged windows, some greedy: a lightly loaded server
        _case("step_b4_v152k", "step", "bf16", 3584, 152064, 32000, 4, 2, 8, greedy=0.25, entries=20000, max_len=4),
        # the batch the headline metric is quoted on: 16 sequences of 8 drafted tokens, 128256-id target
        _case("step_b16_v128k", "step", "bf16", 4096, 128256, 32000, 16, 8, 8, temperature=0.7, entries=50000, max_len=5),
        # the same batch size against a target with a quarter of the vocabulary
        _case("step_b16_v32k", "step", "bf16", 4096, 32000, 32000, 16, 3, 5, temperature=0.7),
        # adaptive (ragged) windows, half of the sequences greedy: a busy server
        _case("step_b64_v152k", "step", "bf16", 3584, 152064, 32000, 64, 1, 10, greedy=0.5, entries=50000, max_len=6),
        # the largest batch: 1024 verified rows, bound by the matrix cores
        _case("step_b128_v128k", "step", "bf16", 4096, 128256, 32000, 128, 7, 7, temperature=0.7, entries=50000, max_len=5),
        # a mid-size fp32 model end to end
        _case("step_f32_b16_v32k", "step", "f32", 1024, 32000, 8000, 16, 3, 3, entries=2000, max_len=4),
        # the caller projects the hidden states itself: many short windows, a vocabulary of odd size
        _case("logits_b300_v32003", "logits", "bf16", 64, 32003, 8000, 300, 3, 3, entries=2000, max_len=4),
        # the drafter's loss on the headline batch
        _case("loss_b16_v128k", "loss", "bf16", 4096, 128256, 32000, 16, 8, 8, temperature=0.7, entries=50000, max_len=5),
        # the stop rule and the acceptance head's loss value on a busy server's batch
        _case("adapt_b64", "adapt", "f32", 8, 16, 16, 64, 1, 10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    call = rng.choice(["step", "step", "step", "step", "step", "step_f32", "logits", "loss", "adapt", "iteration"])
    greedy = rng.choice([0.0, 0.0, 0.3, 0.5])
    temperature = rng.choice([1.0, 0.7, 0.5])
    k_max = rng.randint(1, 10)
    k_min = rng.choice([k_max, rng.randint(1, k_max)])
    if call == "adapt":
        k_max = _log_int(rng, 1, 63)
        return _case(None, "adapt", "f32", 8, 16, 16, _log_int(rng, 1, 512), rng.randint(1, k_max), k_max)
    max_len = rng.randint(2, 6)
    V_d = _log_int(rng, 2000, 32000)
    common = dict(temperature=temperature, greedy=greedy, max_len=max_len)
    if call == "step_f32":
        V_t = _log_int(rng, 500, 32000)
        B = _log_int(rng, 1, 16)
        return _case(None, "step", "f32", 8 * _log_int(rng, 8, 128), V_t, min(V_d, V_t), B, min(k_min, 5), min(k_max, 5),
                     entries=_log_int(rng, 16, V_t // 8), **common)
    V_t = _log_int(rng, 4096, 152064)
    V_d = min(V_d, V_t)
    common["entries"] = min(_log_int(rng, 100, 50000), V_t // 8)
    if call == "logits":
        B = max(1, min(_log_int(rng, 1, 300), 100_000_000 // V_t // (k_max + 1)))
        return _case(None, "logits", rng.choice(["bf16", "bf16", "f32"]), 64, V_t, V_d, B, k_min, k_max, **common)
    d = 8 * _log_int(rng, 64, 512)
    if call == "iteration":
        return _case(None, "iteration", "bf16", d, V_t, V_d, _log_int(rng, 1, 8), k_min, k_max, **common)
    B = max(1, min(_log_int(rng, 1, 256 if call == "step" else 48), 1024 // (k_max + 1)))
    if call == "loss":
        common["greedy"] = min(greedy, 0.3)
        common.update(qprime=rng.random() < 0.3, approx_kl=rng.random() < 0.3)
    return _case(None, call, "bf16", d, V_t, V_d, B, k_min, k_max, **common)


def _lengths(case):
    """Drafted tokens per sequence: part of the case, not of the seed."""
    rng = np.random.default_rng([case["B"], case["k_min"], case["k_max"]])
    return rng.integers(case["k_min"], case["k_max"] + 1, size=case["B"]).astype(np.int32)


# ------------------------------------------------------------------------------------------------ inputs
def _ngrams(rng, V_d, n, max_len, targets_from):
    """n cache entries in CSR form: keys of 2..max_len draft ids with a long-tailed use, target ids of `targets_from`."""
    lens = rng.integers(2, max_len + 1, size=n)
    key_off = np.zeros(n + 1, np.int32)
    key_off[1:] = np.cumsum(lens)
    cdf = np.cumsum(np.arange(1, V_d + 1, dtype=np.float64) ** -1.1)
    rank = np.searchsorted(cdf, rng.random(int(key_off[-1])) * cdf[-1], side="right")
    key_ids = rng.permutation(V_d)[np.minimum(rank, V_d - 1)].astype(np.int32)
    return key_off, key_ids, rng.choice(targets_from, size=n).astype(np.int32)


def _translate(ids, dmap, table, max_len):
    """The window's target tokens, left to right: (target id, first draft position, draft tokens covered)."""
    got, s = [], 0
    while s < len(ids):
        L = next((n for n in range(min(max_len, len(ids) - s), 1, -1) if ids[s:s + n] in table), 1)
        t = table[ids[s:s + L]] if L > 1 else int(dmap[ids[s]])
        if t < 0:
            break
        got.append((t, s, L))
        s += L
    return got


def _inputs(case, seed):
    """All inputs of one batch: small ones as numpy arrays, tensors on the GPU.  `tokens[b]` is the translated window."""
    V_t, V_d, B, d = case["V_t"], case["V_d"], case["B"], case["d"]
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    rng = np.random.default_rng([seed, 7])
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    normal = lambda *shape: torch.randn(*shape, generator=gen, device=DEVICE)  # noqa: E731
    k = _lengths(case)
    row_off = np.zeros(B + 1, np.int32)
    row_off[1:] = np.cumsum(k + 1)
    M, K = int(row_off[-1]), int(k.sum())
    T = np.full(B, case["temperature"], np.float32)
    T[rng.permutation(B)[:int(round(case["greedy"] * B))]] = 0.0
    x = {"k": k, "row_off": row_off, "M": M, "K": K, "T": T, "seed": seed}
    if V_d == V_t:                               # one vocabulary, 2 % of the ids exchanged among themselves
        dmap = np.arange(V_d, dtype=np.int32)
        moved = rng.choice(V_d, size=V_d // 50, replace=False)
        dmap[moved] = moved[rng.permutation(moved.size)]
    else:
        dmap = np.full(V_d, -1, np.int32)
        n = min(int(0.93 * V_d), int(0.8 * V_t))
        dmap[rng.choice(V_d, size=n, replace=False)] = rng.choice(V_t, size=n, replace=False)
    unshared = np.setdiff1d(np.arange(V_t), dmap)
    if case["entries"]:
        x["ngrams"] = _ngrams(rng, V_d, case["entries"], case["max_len"], unshared if unshared.size else np.arange(V_t))
    else:
        x["ngrams"] = (np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32))
    if case["call"] == "iteration":              # what later iterations find: more than the cache holds, so that it evicts
        x["found"] = _ngrams(rng, V_d, case["entries"] + 4000, case["max_len"], unshared if unshared.size else np.arange(V_t))
    key_off, key_ids, targets = x["ngrams"]
    keys = key_ids.tolist()
    entries = [tuple(keys[key_off[e]:key_off[e + 1]]) for e in range(targets.size)]
    table = dict(zip(entries, targets.tolist()))

    # drafted ids: sampled from the drafter's softmax (Gumbel maximum), with cache keys planted over part of the windows
    zq = (SIGMA_Q * normal(K, V_d)).to(dtype)
    Td = torch.from_numpy(np.repeat(T, k)).to(DEVICE)[:, None]
    noise = -torch.log(torch.empty(K, V_d, device=DEVICE).exponential_(generator=gen))
    ids = torch.argmax(zq.float() + Td * noise, 1).cpu().numpy().astype(np.int32)
    del noise
    mean_len = 0.5 * (2 + case["max_len"])
    start = COVER / (mean_len * (1.0 - COVER) + COVER) if entries else 0.0
    tokens, bump, agree = [], [], []
    for b in range(B):
        q0, r0, s = int(row_off[b]) - b, int(row_off[b]), 0
        while s < k[b]:
            key = entries[rng.integers(len(entries))] if entries and rng.random() < start else ()
            if key and s + len(key) <= k[b]:
                ids[q0 + s:q0 + s + len(key)] = key
                s += len(key)
            else:
                s += 1
        got = _translate(tuple(ids[q0:q0 + k[b]].tolist()), dmap, table, case["max_len"])
        tokens.append(got)
        t_b = float(T[b]) or 1.0
        for j, (t, s, L) in enumerate(got):
            if rng.random() >= ALIGN:
                continue
            agree.append((r0 + j, t, t_b, rng.uniform(-2.0, 3.0)))
            if L == 1:
                bump.append((q0 + s, int(ids[q0 + s]), t_b * (math.log(V_d) + 0.5 * (SIGMA_Q / t_b) ** 2 + rng.uniform(-2.0, 2.0))))
    if bump:
        rows, cols, vals = (torch.tensor(v, device=DEVICE) for v in zip(*bump))
        zq[rows, cols] = vals.to(dtype)
    x.update(dmap=dmap, table=table, tokens=tokens, draft_logits=zq, draft_ids=ids)

    # target side: the rows of agreeable positions favour the proposed token
    sigma_z = SIGMA_W * math.sqrt(4096 if case["call"] == "logits" else d)
    if agree:
        rows, toks, temps, lifts = zip(*agree)
        rows, toks = torch.tensor(rows, device=DEVICE), torch.tensor(toks, device=DEVICE)
        want = torch.tensor([t * (math.log(V_t) + 0.5 * (sigma_z / t) ** 2 + u) for t, u in zip(temps, lifts)], device=DEVICE)
    if case["call"] == "logits":
        Z = sigma_z * normal(M, V_t)
        if agree:
            Z[rows, toks] = want
        x["target_logits"] = Z
        x["W"] = torch.zeros(d, V_t, dtype=dtype, device=DEVICE)
        return x
    W = torch.empty(d, V_t, dtype=dtype, device=DEVICE)
    for r in range(0, d, 512):
        W[r:r + 512] = (SIGMA_W * normal(min(512, d - r), V_t)).to(dtype)
    hidden = normal(M, d)
    if agree:
        cols = W[:, toks].float()
        hidden[rows] = (cols * (want / cols.square().sum(0))).t() + 0.3 * hidden[rows]
    x["W"], x["hidden"] = W, hidden.to(dtype)
    return x


class _DeviceView:
    """A tensor's worth of the context's workspace; keeps the context alive as long as a tensor looks at it."""

    def __init__(self, owner, ptr, shape, typestr, strides=None):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": shape, "typestr": typestr, "data": (ptr, False), "strides": strides, "version": 2}


def _workspace(v, M, K, V_t, with_logits):
    """Tensors that look at the row statistics (and logits) which a step leaves in the context's workspace."""
    w = ot.ot_verify_workspace(v.ctx)
    look = lambda *a: torch.as_tensor(_DeviceView(v, *a), device=DEVICE)  # noqa: E731
    out = {"row_max": look(w.row_max, (M,), "<f4"), "row_sumexp": look(w.row_sumexp, (M,), "<f8"),
           "draft_row_max": look(w.draft_row_max, (K,), "<f4"), "draft_row_sumexp": look(w.draft_row_sumexp, (K,), "<f8")}
    if with_logits:
        out["logits"] = look(w.logits, (M, V_t), "<f4", (4 * int(w.ld_logits), 4))
    return out


def _adapt_inputs(case, seed):
    rng = np.random.default_rng([seed, 11])
    k = _lengths(case)
    row_off = np.zeros(case["B"] + 1, np.int32)
    row_off[1:] = np.cumsum(k + 1)
    M = int(row_off[-1])
    return {"k": k, "row_off": row_off, "M": M, "head_logits": (2.0 * rng.standard_normal(M) + 2.0).astype(np.float32),
            "labels": np.clip(rng.uniform(-0.2, 1.4, M), 0.0, 1.0).astype(np.float32)}


GAMMA, W_ACCEPT, W_REJECT = 0.7, 1.0, 6.0


def prepare(case, seed):
    put = lambda a: torch.from_numpy(a).to(DEVICE)  # noqa: E731
    call, B = case["call"], case["B"]
    if call == "adapt":
        x = _adapt_inputs(case, seed)
        v = Verifier(d=case["d"], V_t=case["V_t"], V_d=case["V_d"], dtype="f32", W=torch.zeros(case["d"], case["V_t"], device=DEVICE),
                     direct_map=np.arange(case["V_d"], dtype=np.int32), max_batch=B, max_k=case["k_max"])
        new = lambda n, t: torch.empty(n, dtype=t, device=DEVICE)  # noqa: E731
        out = {"p_accept": new(x["M"], torch.float32), "p_any_reject": new(x["M"], torch.float32), "n_keep": new(B, torch.int32),
               "bce": new(3, torch.float64)}
        args = {"B": B, "gamma": GAMMA, "w_accept": W_ACCEPT, "w_reject": W_REJECT, "row_off": put(x["row_off"]),
                "row_off_host": x["row_off"], "head_logits": put(x["head_logits"]), "labels": put(x["labels"])}
        return {"call": call, "v": v, "args": args, "out": out}
    x = _inputs(case, seed)
    v = Verifier(d=case["d"], V_t=case["V_t"], V_d=case["V_d"], dtype=case["dtype"], W=x["W"], direct_map=x["dmap"], max_batch=B,
                 max_k=case["k_max"], max_ngram_len=case["max_len"])
    state = {"call": call, "v": v}
    if call == "iteration":
        v.cache = ot.ot_ngram_cache_create(v.ctx, case["entries"], ot.OT_EVICT_LRU)
        ot.ot_ngram_cache_insert(v.cache, *x["ngrams"])
        key_off, key_ids, targets = x["found"]
        state["turn"], state["found"] = 0, []
        for e in range(0, targets.size - 7, 8):      # eight n-grams an iteration
            o = key_off[e:e + 9]
            state["found"].append((o - o[0], key_ids[o[0]:o[-1]], targets[e:e + 8]))
    else:
        v.set_cache(*x["ngrams"])
    state["inp"] = {"B": B, "M": x["M"], "K": x["K"], "step": 3, "seed": seed, "row_off_host": x["row_off"], "row_off": put(x["row_off"]),
                    "hidden": x.get("hidden"), "target_logits": x.get("target_logits"), "draft_logits": x["draft_logits"],
                    "draft_ids": put(x["draft_ids"]), "temperature": put(x["T"]), "draft_temperature": None,
                    "seq_id": torch.arange(B, dtype=torch.int64, device=DEVICE), "out": v.alloc_outputs(B, x["M"])}
    if call == "loss":
        v.step(state["inp"])
        state["loss"] = {"lam": 0.2, "lambda_mode": ot.OT_LAMBDA_TARGET_PROB if case["approx_kl"] else ot.OT_LAMBDA_FIXED,
                         "ngram_term": ot.OT_NGRAM_TERM_APPROX_KL if case["approx_kl"] else ot.OT_NGRAM_TERM_NLL,
                         "with_qprime": case["qprime"]}
        v.distill_loss(state["inp"], **state["loss"])
        state["out"] = state["inp"]["loss_buffers", max(x["M"], 1), case["qprime"]]
    else:
        state["out"] = dict(state["inp"]["out"], **_workspace(v, x["M"], x["K"], case["V_t"], call != "logits"))
    return state


def run(state):
    v, call = state["v"], state["call"]
    if call == "adapt":
        ot.ot_adaptive_drafting(v.ctx, **state["args"], **state["out"])
    elif call == "loss":
        v.distill_loss(state["inp"], sync=False, **state["loss"])
    else:
        v.step(state["inp"], from_logits=call == "logits")
        if call == "iteration":
            found = state["found"][state["turn"] % len(state["found"])]
            state["turn"] += 1
            return dict(state["out"], n_evicted=ot.ot_ngram_cache_insert(v.cache, *found))
    return state["out"]


# ------------------------------------------------------------------------------------------------ what a pass costs
def work(case):
    """Inputs read once, outputs written once; operations of the projection, or a few per logit where there is none."""
    k = _lengths(case)
    K, M, V_t, V_d, d = int(k.sum()), int(k.sum()) + case["B"], case["V_t"], case["V_d"], case["d"]
    esz = 2 if case["dtype"] == "bf16" else 4
    if case["call"] == "adapt":
        return {"bytes": 16.0 * M + 8.0 * case["B"], "flops": 40.0 * K}
    if case["call"] == "logits":
        return {"bytes": 4.0 * M * V_t + esz * K * V_d + 4.0 * V_t, "flops": 4.0 * (M * V_t + K * V_d)}
    if case["call"] == "loss":
        # tokens with a KL term: the windows' positions less those that n-grams cover (all tokens with the approximate KL)
        rows = K * (1.0 - COVER * (0.5 if case["approx_kl"] else 1.0) * (case["entries"] > 0)) * (1.0 - case["greedy"])
        return {"bytes": rows * (4.0 * V_t + esz * V_d) + 4.0 * V_t + (4.0 * M * V_t if case["qprime"] else 0.0), "flops": 12.0 * rows * V_t}
    return {"bytes": float(esz) * (d * V_t + M * d + K * V_d) + 4.0 * M * V_t + 4.0 * V_t, "flops": 2.0 * M * d * V_t}


def tolerance(case):
    """Sums of a few thousand binary32 terms; whole values may differ where a draw falls onto the edge of two tokens."""
    if case["call"] == "adapt":
        return {"rel": 1e-6}
    if case["call"] == "logits":
        return {"rel": 2e-6, "max": 1e-5, "differ": 0.004}
    return {"rel": 1e-5, "max": 4e-4, "differ": 0.01}


# ------------------------------------------------------------------------------------------------ in 64 bits
def _row_stats(z, T):
    """(max, sum exp((z - max) / T)) of rows z; T == 0 rows at temperature 1."""
    mx = z.max(1).values
    return mx, torch.exp((z - mx[:, None]) / torch.where(T > 0, T, 1.0)[:, None]).sum(1)


def _exact_loss(case, x, Z, T_rows, T_draft):
    M, V_t = x["M"], case["V_t"]
    mx, S = _row_stats(Z, T_rows)
    zq = x["draft_logits"].double()
    mxq, Sq = _row_stats(zq, T_draft)
    dmap = torch.from_numpy(x["dmap"]).to(DEVICE).long()
    mapped = dmap >= 0
    out = {n: torch.zeros(M, dtype=torch.float64) for n in ("kl", "nll", "weight")}
    qp = torch.zeros(M, V_t, dtype=torch.float32, device=DEVICE) if case["qprime"] else None
    sums, counts = [0.0, 0.0], [0, 0]
    for b, got in enumerate(x["tokens"]):
        r0, q0, T = int(x["row_off"][b]), int(x["row_off"][b]) - b, float(x["T"][b])
        if T <= 0:
            continue
        for j, (t, s, L) in enumerate(got):
            r = r0 + j
            lq_row = (zq[q0 + s] - mxq[q0 + s]) / T - torch.log(Sq[q0 + s])
            lq = torch.full((V_t,), -math.inf, dtype=torch.float64, device=DEVICE)
            lq[dmap[mapped]] = lq_row[mapped]
            if L > 1:
                logs = [float((zq[q0 + s + i, int(x["draft_ids"][q0 + s + i])] - mxq[q0 + s + i]) / T - torch.log(Sq[q0 + s + i])) for i in range(L)]
                first = int(x["dmap"][x["draft_ids"][q0 + s]])
                if first >= 0:
                    rest = math.exp(logs[0]) - math.exp(sum(logs))
                    lq[first] = math.log(rest) if rest > 0 else -math.inf
                lq[t] = sum(logs)
                out["nll"][r] = -sum(logs)
                lp_t = float((Z[r, t] - mx[r]) / T - torch.log(S[r]))
                out["weight"][r] = math.exp(lp_t) if case["approx_kl"] else float(np.float32(0.2))
            q = torch.exp(lq)
            if qp is not None:
                qp[r] = q.float()
            if L == 1 or case["approx_kl"]:
                lp = (Z[r] - mx[r]) / T - torch.log(S[r])
                out["kl"][r] = float(torch.where(q > 0, q * (lq - lp), 0.0).sum())
            if L == 1:
                sums[0] += float(out["kl"][r])
                counts[0] += 1
            else:
                sums[1] += float(out["weight"][r] * (out["kl"][r] if case["approx_kl"] else out["nll"][r]))
                counts[1] += L
    out["totals"] = torch.tensor(sums + counts + [sum(sums) / max(1, sum(counts))], dtype=torch.float64)
    out["kind"] = None
    if qp is not None:
        out["qprime"] = qp
    return out


def exact(case, seed):
    if case["call"] == "adapt":
        x = _adapt_inputs(case, seed)
        a, lab = x["head_logits"].astype(np.float64), x["labels"].astype(np.float64)
        p, rej, total, n = np.zeros(x["M"]), np.zeros(x["M"]), 0.0, int(x["k"].sum())
        for b, k in enumerate(x["k"]):
            at = slice(int(x["row_off"][b]), int(x["row_off"][b]) + int(k))
            p[at] = 1.0 / (1.0 + np.exp(-a[at]))
            rej[at] = 1.0 - np.cumprod(p[at])
            cost = W_ACCEPT * lab[at] * np.logaddexp(0.0, -a[at]) + W_REJECT * (1.0 - lab[at]) * np.logaddexp(0.0, a[at])
            total += float(cost.sum())
        return {"p_accept": p, "p_any_reject": rej, "n_keep": None, "bce": np.array([total, n, total / max(1, n)])}
    x = _inputs(case, seed)
    if case["call"] == "logits":
        Z = x["target_logits"].double()
    else:
        Z = torch.empty(x["M"], case["V_t"], dtype=torch.float64, device=DEVICE)
        hidden = x["hidden"].double()
        for c in range(0, case["V_t"], 16384):
            Z[:, c:c + 16384] = hidden @ x["W"][:, c:c + 16384].double()
    T = torch.from_numpy(x["T"]).to(DEVICE).double()
    k = torch.from_numpy(x["k"]).to(DEVICE).long()
    T_rows, T_draft = torch.repeat_interleave(T, k + 1), torch.repeat_interleave(T, k)
    if case["call"] == "loss":
        return _exact_loss(case, x, Z, T_rows, T_draft)
    mx, S = _row_stats(Z, T_rows)
    zq = x["draft_logits"].double()
    mxq, Sq = _row_stats(zq, T_draft)
    ids = torch.from_numpy(x["draft_ids"]).to(DEVICE).long()
    lq = ((zq.gather(1, ids[:, None])[:, 0] - mxq) / torch.where(T_draft > 0, T_draft, 1.0) - torch.log(Sq)).cpu().numpy()
    lq_greedy = np.where((zq.argmax(1) == ids).cpu().numpy(), 0.0, -np.inf)
    best = Z.argmax(1).cpu().numpy()
    p_tok, q_tok, ratio = (np.zeros(x["M"]) for _ in range(3))
    rows, toks = [], []
    for b, got in enumerate(x["tokens"]):
        r0, q0 = int(x["row_off"][b]), int(x["row_off"][b]) - b
        for j, (t, s, L) in enumerate(got):
            rows.append(r0 + j)
            toks.append(t)
            q_tok[r0 + j] = math.exp((lq if x["T"][b] > 0 else lq_greedy)[q0 + s:q0 + s + L].sum())
    if rows:
        r, t = torch.tensor(rows, device=DEVICE), torch.tensor(toks, device=DEVICE)
        p = (torch.exp((Z[r, t] - mx[r]) / torch.where(T_rows > 0, T_rows, 1.0)[r]) / S[r]).cpu().numpy()
        greedy = (T_rows <= 0).cpu().numpy()
        for i, (r, t) in enumerate(zip(rows, toks)):
            p_tok[r] = float(best[r] == t) if greedy[r] else p[i]
            ratio[r] = p_tok[r] if greedy[r] else min(1.0, p_tok[r] / q_tok[r]) if q_tok[r] > 0 else float(p_tok[r] > 0)
    out = {n: None for n in ot.OUT_INT_B + ot.OUT_INT_M}
    out.update(p_tok=p_tok, q_tok=q_tok, ratio=ratio, row_max=mx, row_sumexp=S, draft_row_max=mxq, draft_row_sumexp=Sq)
    if case["call"] != "logits":
        out["logits"] = Z
    if case["call"] == "iteration":
        out["n_evicted"] = None
    return out
