"""The work that a user of this framework has it do, as cases that can be timed and checked.

A case is a dict of plain values; `kind` says which public entry points one pass calls:

  step     a decode step of the pool as the rollout loop enqueues it: copris_rollout_apply,
           copris_kv_append, copris_decode_attn, copris_lmhead_logprob, copris_traj_append
  attn     copris_decode_attn of one layer
  sample   copris_lmhead_logprob
  given    copris_lmhead_token_logprob
  prefill  copris_prefill_attn
  batch    what is done with the log-probs of a training batch: copris_traj_gather,
           copris_is_ratio, copris_grpo_surrogate

Lengths are the quantiles of the case's length distribution, in an order that the seed
chooses: the amount of work of a case is fixed, its arrangement is not.
"""
from __future__ import annotations

import math
from statistics import NormalDist

import numpy as np
import torch

from paper_2511_05589_amd import binding as B

DTYPES = {"bf16": (torch.bfloat16, B.COPRIS_BF16, 2), "f32": (torch.float32, B.COPRIS_F32, 4)}


# ---- the cases ---------------------------------------------------------------------------------
def listed():
    c1 = dict(prompt=256, mu=7.0, sigma=1.0, cap=8192)
    c2 = dict(prompt=512, mu=7.5, sigma=1.1, cap=16384)
    return [
        # the smallest pool: a debugging run in fp32, where launches and latency count
        dict(name="step_tiny_f32", kind="step", dtype="f32", C=8, Hq=4, Hkv=2, D=64, page=16, prompt=32, mu=5.0,
             sigma=1.0, cap=512, H=256, V=1024, T=1.0),
        # a whole decode step of a 1.5B-shaped model's last layer and head: an ordinary pool on one GPU
        dict(name="step_c64", kind="step", dtype="bf16", C=64, Hq=12, Hkv=2, D=128, page=16, H=1536, V=151936, T=1.0,
             **c1),
        # decode attention of a 7B-shaped layer, the pool that the headline metric is quoted on
        dict(name="attn_c256", kind="attn", dtype="bf16", C=256, Hq=28, Hkv=4, D=128, page=16, **c2),
        # the long-tail pool: hundreds of short contexts and a few resumed 32k-token trajectories
        dict(name="attn_longtail_c512", kind="attn", dtype="bf16", C=512, Hq=28, Hkv=4, D=128, page=16, prompt=0,
             mu=0.0, sigma=0.0, cap=32768),
        # decode attention of a model with 64-wide heads
        dict(name="attn_d64_c64", kind="attn", dtype="bf16", C=64, Hq=16, Hkv=4, D=64, page=16, **c1),
        # sampling head of the 7B shape at the headline pool
        dict(name="sample_c256", kind="sample", dtype="bf16", C=256, H=3584, V=151936, T=1.0),
        # sampling head with an odd pool that is drained unevenly, an odd vocabulary and the evaluation temperature
        dict(name="sample_c301_odd", kind="sample", dtype="bf16", C=301, H=2048, V=50257, T=0.6),
        # log-probs of the buffered tokens under the new policy: a full micro-batch
        dict(name="given_8192", kind="given", dtype="bf16", M=8192, H=3584, V=151936, T=1.0),
        # ... and the odd-sized rest of a batch
        dict(name="given_777", kind="given", dtype="bf16", M=777, H=1536, V=151936, T=1.0),
        # the start of a stage: sixteen resumed trajectories are re-prefilled together
        dict(name="prefill_16", kind="prefill", dtype="bf16", n=16, Hq=28, Hkv=4, **c2),
        # the middle of a stage: two requests enter and are prefilled, one of them resumed
        dict(name="prefill_2", kind="prefill", dtype="bf16", n=2, Hq=12, Hkv=2, prompt=150, mu=6.0, sigma=1.0, cap=8192),
        # a training batch: the cross-stage ratio, the surrogate and its gradient
        dict(name="batch_256", kind="batch", Bt=256, lo=1024, hi=16384, mask=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_ctx(rng):
    return dict(prompt=_log_int(rng, 32, 1024), mu=rng.uniform(5.0, 7.5), sigma=rng.uniform(0.8, 1.1),
                cap=rng.choice([512, 4096, 8192, 16384]))


def draw(rng):
    kind = rng.choice(["step", "attn", "attn", "sample", "given", "prefill", "batch"])
    while True:
        if kind in ("step", "attn"):
            Hq, Hkv, D = rng.choice([(28, 4, 128), (12, 2, 128), (8, 8, 128), (16, 1, 128), (4, 2, 64), (16, 4, 64),
                                     (6, 2, 64), (14, 2, 64)])
            c = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), C=_log_int(rng, 1, 512), Hq=Hq, Hkv=Hkv,
                     D=D, page=rng.choice([16, 16, 16, 8, 32]), **_draw_ctx(rng))
            kv = sum(_lengths(c)) * Hkv * D * 2 * DTYPES[c["dtype"]][2]
            # pools of the sizes that the configurations have; fp32 is for small runs
            if kv > (2.5e9 if c["dtype"] == "bf16" else 0.2e9):
                continue
            if kind == "step":
                c.update(H=rng.choice([256, 512, 1024, 1536, 3584]), V=_log_int(rng, 1000, 151936), T=rng.choice([1.0, 0.6]))
                if c["dtype"] == "f32" and c["C"] * c["H"] * c["V"] > 64 * 1024 * 32768:
                    continue
            return c
        if kind == "sample":
            return dict(kind=kind, dtype="bf16", C=_log_int(rng, 1, 512), H=rng.choice([256, 512, 1024, 1536, 2048, 3584]),
                        V=_log_int(rng, 4096, 151936), T=rng.choice([1.0, 0.6]))
        if kind == "given":
            return dict(kind=kind, dtype="bf16", M=_log_int(rng, 16, 8192), H=rng.choice([256, 512, 1024, 1536, 2048, 3584]),
                        V=_log_int(rng, 4096, 151936), T=rng.choice([1.0, 0.6]))
        if kind == "prefill":
            Hq, Hkv = rng.choice([(28, 4), (12, 2), (16, 4), (8, 8), (8, 1), (32, 4), (6, 2)])
            c = dict(kind=kind, dtype="bf16", n=_log_int(rng, 1, 24), Hq=Hq, Hkv=Hkv, **_draw_ctx(rng))
            if work(c)["flops"] > 4.4e12:
                continue
            return c
        lo = _log_int(rng, 1, 4096)
        c = dict(kind="batch", Bt=_log_int(rng, 1, 512), lo=lo, hi=lo + _log_int(rng, 1, 16384), mask=rng.random() < 0.5)
        if sum(_lengths(c)) > 2_300_000:
            continue
        return c


def _lengths(case):
    """The lengths of the case's sequences, shortest first."""
    if case["kind"] == "batch":
        n, lo, hi = case["Bt"], case["lo"], case["hi"]
        return [lo + int((hi - lo) * (i + 0.5) / n) for i in range(n)]
    n = case["n"] if case["kind"] == "prefill" else case["C"]
    if case["sigma"] == 0.0:   # the long-tail recipe: 90 % in 256..2048, 8 % in 2048..16384, 2 % at the cap
        n_long, n_mid = round(0.02 * n), round(0.08 * n)
        n_short = n - n_long - n_mid
        return ([256 + int(1792 * (i + 0.5) / n_short) for i in range(n_short)]
                + [2048 + int(14336 * (i + 0.5) / n_mid) for i in range(n_mid)] + [case["cap"]] * n_long)
    z = NormalDist()
    return [case["prompt"] + min(max(round(math.exp(case["mu"] + case["sigma"] * z.inv_cdf((i + 0.5) / n))), 1), case["cap"])
            for i in range(n)]


def work(case):
    """What a pass cannot do without: each input read once, each output written once."""
    kind = case["kind"]
    if kind == "batch":
        n, b = sum(_lengths(case)), case["Bt"]
        # gather: token, log-prob and tag in, token and both sides out; ratio and surrogate: current and one old log-prob
        # (and the mask) in, two values out
        return {"bytes": n * (24 + 2 * (16 + (1 if case["mask"] else 0))) + b * 48, "flops": 10 * n}
    es = DTYPES[case["dtype"]][2]
    if kind in ("sample", "given"):
        m = case["C"] if kind == "sample" else case["M"]
        return {"bytes": (m + case["V"]) * case["H"] * es + m * 24, "flops": 2 * m * case["H"] * case["V"]}
    if kind == "prefill":
        lens, Hq, Hkv, D = _lengths(case), case["Hq"], case["Hkv"], 128
        t = sum(lens)
        return {"bytes": t * (2 * Hq * D + 4 * Hkv * D) * es + t * Hq * 4, "flops": 4 * Hq * D * sum(n * (n + 1) // 2 for n in lens)}
    C, Hq, Hkv, D = case["C"], case["Hq"], case["Hkv"], case["D"]
    t = sum(_lengths(case))
    w = {"bytes": t * 2 * Hkv * D * es + 4 * (t // case["page"] + C) + 2 * C * Hq * D * es + C * Hq * 4, "flops": 4 * t * Hq * D}
    if kind == "step":
        w["bytes"] += 4 * C * Hkv * D * es + (C + case["V"]) * case["H"] * es + C * 64
        w["flops"] += 2 * C * case["H"] * case["V"]
    return w


def tolerance(case):
    if case["kind"] == "batch":
        return {"rel": 1e-5}                     # fp32 exponentials and sums of thousands of terms
    if case["kind"] in ("sample", "given") or case["dtype"] == "f32":
        # fp32 sums over the hidden dimension and the vocabulary; a token may change on a tie
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}
    # attention in bf16: the weights and the result are rounded to 8 bits
    return {"rel": 1e-2, "max": 0.1, "differ": 0.005}


# ---- inputs ------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)


def _normal(g, shape, dtype, std=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=DTYPES[dtype][0])
    return x.mul_(std) if std != 1.0 else x


def _shuffled_lengths(case, seed):
    return np.random.default_rng(int(seed)).permutation(np.array(_lengths(case), dtype=np.int64)).astype(np.int32)


def _pages(g, lens, page):
    """A block table over physical pages in random order, a quarter of them free."""
    npg = torch.from_numpy((lens.astype(np.int64) + page - 1) // page).cuda()
    used, width = int(npg.sum()), int(npg.max())
    num_pages = used + used // 4 + 1
    bt = torch.full((len(lens), width), -1, dtype=torch.int32, device="cuda")
    own = torch.arange(width, device="cuda")[None, :] < npg[:, None]
    bt[own] = torch.randperm(num_pages, generator=g, device="cuda")[:used].to(torch.int32)
    return bt, num_pages


def _empty(*shape, dtype=torch.float32):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _inputs(case, seed):
    """The inputs of a pass, from the seed alone."""
    g, kind, s = _gen(seed), case["kind"], {}
    if kind in ("step", "attn"):
        C, Hq, Hkv, D, dt = case["C"], case["Hq"], case["Hkv"], case["D"], case["dtype"]
        lens = _shuffled_lengths(case, seed)
        s["lens"], s["ctx_len"] = lens, torch.from_numpy(lens).cuda()
        s["block_table"], n = _pages(g, lens, case["page"])
        s["q"] = _normal(g, (C, Hq, D), dt)
        s["k_cache"], s["v_cache"] = (_normal(g, (n, Hkv, case["page"], D), dt) for _ in "kv")
        if kind == "step":
            s["k_new"], s["v_new"] = (_normal(g, (C, Hkv, D), dt) for _ in "kv")
            # the pool's occupants and where each of them stands; set by commands, as the manager does at a stage's start
            s["step"] = torch.from_numpy(np.maximum(lens - case["prompt"] - 1, 0).astype(np.int32)).cuda()
            s["seq_id"] = torch.randperm(C, generator=g, device="cuda")
            slot = torch.arange(C, device="cuda", dtype=torch.int32)
            s["cmds"] = torch.stack([slot, s["seq_id"].to(torch.int32), s["ctx_len"], s["step"]], 1).reshape(-1).contiguous()
    if kind in ("step", "sample", "given"):
        m = case["M"] if kind == "given" else case["C"]
        s["hidden"] = _normal(g, (m, case["H"]), case["dtype"])
        s["weight"] = _normal(g, (case["V"], case["H"]), case["dtype"], std=0.02)
        s["seed"] = 0x5EED0000 + int(seed)
        if kind == "sample":
            s["seq_id"] = torch.randint(0, 1 << 40, (m,), generator=g, device="cuda")
            s["step"] = torch.randint(0, 16384, (m,), generator=g, device="cuda", dtype=torch.int32)
        if kind == "given":
            s["tokens"] = torch.randint(0, case["V"], (m,), generator=g, device="cuda", dtype=torch.int32)
    if kind == "prefill":
        lens = _shuffled_lengths(case, seed)
        T, Hq, Hkv, D, dt = int(lens.sum()), case["Hq"], case["Hkv"], 128, case["dtype"]
        s["lens"], s["max_seqlen"] = lens, int(lens.max())
        s["cu"] = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        s["block_table"], s["num_pages"] = _pages(g, lens, 16)
        s["q"] = _normal(g, (T, Hq, D), dt)
        s["k"], s["v"] = (_normal(g, (T, Hkv, D), dt) for _ in "kv")
    if kind == "batch":
        lens = _shuffled_lengths(case, seed)
        b, N = len(lens), int(lens.sum())
        s["lens"] = lens
        s["cu"] = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        rows = b + b // 2 + 1                               # the buffer holds other trajectories too
        s["max_resp"] = int(lens.max())
        s["traj"] = torch.randperm(rows, generator=g, device="cuda")[:b].to(torch.int32)
        s["buf_token"] = torch.randint(0, 151936, (rows, s["max_resp"]), generator=g, device="cuda", dtype=torch.int32)
        s["buf_logp"] = torch.empty(rows, s["max_resp"], device="cuda").exponential_(generator=g).neg_()
        # a random stage boundary in every row: earlier tokens are tagged with the stage before this one
        share = torch.rand(rows, 1, generator=g, device="cuda")
        length = torch.full((rows, 1), s["max_resp"], device="cuda")
        length[s["traj"].long(), 0] = torch.from_numpy(lens.astype(np.int64)).cuda()
        s["boundary"] = (share * (length + 1)).long().clamp(max=s["max_resp"])
        s["buf_tag"] = torch.where(torch.arange(s["max_resp"], device="cuda")[None, :] < s["boundary"], 6, 7).to(torch.int32)
        # the current policy's log-probs: the buffered ones and a little drift
        base = torch.cat([s["buf_logp"][t, :n] for t, n in zip(s["traj"].tolist(), lens.tolist())])
        s["logp_cur"] = base + 0.05 * torch.randn(N, generator=g, device="cuda")
        s["mask"] = (torch.rand(N, generator=g, device="cuda") >= 0.01).to(torch.uint8) if case["mask"] else None
        s["adv"] = torch.randn(b, generator=g, device="cuda")
    return s


def prepare(case, seed):
    """Inputs, and the result buffers and workspaces that a program keeps beside them."""
    s, kind = _inputs(case, seed), case["kind"]
    s["case"] = case
    if kind in ("step", "attn"):
        C, Hq, Hkv, D = case["C"], case["Hq"], case["Hkv"], case["D"]
        s["out"], s["lse"] = torch.empty_like(s["q"]), _empty(C, Hq)
        s["ws"] = _bytes(B.decode_attn_workspace_bytes(C, Hq, Hkv, D, case["page"], s["block_table"].shape[1]))
    if kind in ("step", "sample"):
        m = case["C"]
        s["token"], s["logprob"], s["lm_lse"] = _empty(m, dtype=torch.int32), _empty(m), _empty(m)
        s["lm_ws"] = _bytes(B.lmhead_logprob_workspace_bytes(m, case["H"], case["V"]))
    if kind == "step":
        s["pool_seq"] = torch.full((case["C"],), -1, dtype=torch.int64, device="cuda")
        s["pool_ctx"] = torch.zeros(case["C"], dtype=torch.int32, device="cuda")
        s["pool_step"] = torch.zeros(case["C"], dtype=torch.int32, device="cuda")
        rows = (case["C"], case["cap"])
        s["buf_token"] = torch.full(rows, -1, dtype=torch.int32, device="cuda")
        s["buf_logp"] = torch.zeros(rows, device="cuda")
        s["buf_tag"] = torch.full(rows, -1, dtype=torch.int32, device="cuda")
    if kind == "given":
        m = case["M"]
        s["logprob"], s["lse"] = _empty(m), _empty(m)
        s["ws"] = _bytes(B.lmhead_token_logprob_workspace_bytes(m, case["H"], case["V"], DTYPES[case["dtype"]][1]))
    if kind == "prefill":
        shape = (s["num_pages"], case["Hkv"], 16, 128)
        s["k_cache"], s["v_cache"] = (torch.zeros(shape, dtype=s["q"].dtype, device="cuda") for _ in "kv")
        s["out"], s["lse"] = torch.empty_like(s["q"]), _empty(s["q"].shape[0], case["Hq"])
    if kind == "batch":
        N, b = s["logp_cur"].numel(), case["Bt"]
        for name in ("logp_buf", "logp_roll", "ratio", "clipped", "surr", "grad"):
            s[name] = _empty(N)
        s["tokens"] = _empty(N, dtype=torch.int32)
        for name in ("seq_sum", "seq_surr"):
            s[name] = _empty(b)
        for name in ("split", "seq_cnt", "seq_nclip", "seq_cnt2"):
            s[name] = _empty(b, dtype=torch.int32)
        s["objective"] = _empty(2)
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "batch":
        B.traj_gather(s["buf_token"], s["buf_logp"], s["buf_tag"], s["traj"], s["cu"], 7, s["tokens"], s["logp_buf"],
                      s["logp_roll"], s["split"])
        B.is_ratio(s["logp_cur"], s["logp_buf"], s["logp_roll"], s["cu"], s["split"], s["mask"], s["ratio"], s["clipped"],
                   s["seq_sum"], s["seq_cnt"], s["seq_nclip"], eps_low=0.2, eps_high=0.28)
        B.grpo_surrogate(s["logp_cur"], s["logp_buf"], s["logp_roll"], s["cu"], s["split"], s["mask"], s["adv"], s["surr"],
                         s["grad"], s["seq_surr"], s["seq_cnt2"], s["objective"], eps_low=0.2, eps_high=0.28)
        return {k: s[k] for k in ("tokens", "logp_buf", "logp_roll", "split", "ratio", "clipped", "seq_sum", "seq_cnt",
                                  "seq_nclip", "surr", "grad", "seq_surr", "seq_cnt2", "objective")}
    dt = DTYPES[case["dtype"]][1]
    if kind == "given":
        B.lmhead_token_logprob(s["hidden"], s["weight"], s["tokens"], s["logprob"], s["lse"], s["ws"], temperature=case["T"],
                               dtype=dt)
        return {"logprob": s["logprob"], "lse": s["lse"]}
    if kind == "sample":
        B.lmhead_logprob(s["hidden"], s["weight"], s["seq_id"], s["step"], s["token"], s["logprob"], s["lm_lse"], s["lm_ws"],
                         seed=s["seed"], temperature=case["T"], dtype=dt)
        return {"token": s["token"], "logprob": s["logprob"], "lse": s["lm_lse"]}
    if kind == "prefill":
        B.prefill_attn(s["q"], s["k"], s["v"], s["cu"], s["block_table"], s["k_cache"], s["v_cache"], s["out"], s["lse"],
                       max_seqlen=s["max_seqlen"], scale=128 ** -0.5, dtype=dt)
        return {"out": s["out"], "lse": s["lse"], "k_cache": s["k_cache"], "v_cache": s["v_cache"]}
    scale = case["D"] ** -0.5
    if kind == "attn":
        B.decode_attn(s["q"], s["k_cache"], s["v_cache"], s["block_table"], s["ctx_len"], s["out"], s["lse"], s["ws"],
                      scale=scale, dtype=dt)
        return {"out": s["out"], "lse": s["lse"]}
    B.rollout_apply(s["cmds"], case["C"], 0, s["pool_seq"], s["pool_ctx"], s["pool_step"], s["block_table"])
    B.kv_append(s["k_new"], s["v_new"], s["block_table"], s["pool_ctx"], s["k_cache"], s["v_cache"], dtype=dt)
    B.decode_attn(s["q"], s["k_cache"], s["v_cache"], s["block_table"], s["pool_ctx"], s["out"], s["lse"], s["ws"],
                  scale=scale, dtype=dt)
    B.lmhead_logprob(s["hidden"], s["weight"], s["pool_seq"], s["pool_step"], s["token"], s["logprob"], s["lm_lse"], s["lm_ws"],
                     seed=s["seed"], temperature=case["T"], dtype=dt)
    B.traj_append(s["token"], s["logprob"], s["pool_seq"], s["pool_step"], s["pool_ctx"], 3, s["buf_token"], s["buf_logp"],
                  s["buf_tag"])
    return {k: s[k] for k in ("out", "lse", "token", "logprob", "lm_lse", "pool_seq", "pool_ctx", "pool_step", "k_cache",
                              "v_cache", "buf_token", "buf_logp", "buf_tag")}


# ---- the same in 64 bits, in plain torch ---------------------------------------------------------
def _softmax_attn(q, k, v, scale, causal):
    """q [n, Hq, D], k and v [m, Hkv, D] in float64 (n = m where causal): out [n, Hq, D], lse [n, Hq]."""
    n, Hq, D = q.shape
    m, Hkv, _ = k.shape
    kt, vv = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
    g, outs, lses = Hq // Hkv, [], []
    for r in range(0, n, 512):
        qq = q[r:r + 512]
        w = qq.shape[0]
        seen = r + w if causal else m
        sc = torch.matmul(qq.reshape(w, Hkv, g, D).permute(1, 2, 0, 3).reshape(Hkv, g * w, D).contiguous(),
                          kt[:, :, :seen].contiguous()).mul_(scale).view(Hkv, g, w, seen)
        if causal:
            at = torch.arange(r, r + w, device=q.device)
            sc.masked_fill_(torch.arange(seen, device=q.device)[None, :] > at[:, None], -math.inf)
        lse = torch.logsumexp(sc, -1)
        o = torch.matmul(sc.sub_(lse[..., None]).exp_().view(Hkv, g * w, seen), vv[:, :seen].contiguous())
        outs.append(o.view(Hkv, g, w, D).permute(2, 0, 1, 3).reshape(w, Hq, D))
        lses.append(lse.permute(2, 0, 1).reshape(w, Hq))
    return torch.cat(outs), torch.cat(lses)


def _paged_attn(s, case):
    outs, lses = [], []
    for i, n in enumerate(s["lens"].tolist()):
        pages = s["block_table"][i, :(n + case["page"] - 1) // case["page"]].long()
        k, v = (s[x][pages].permute(0, 2, 1, 3).reshape(-1, case["Hkv"], case["D"])[:n].double() for x in ("k_cache", "v_cache"))
        o, l = _softmax_attn(s["q"][i:i + 1].double(), k, v, case["D"] ** -0.5, False)
        outs.append(o)
        lses.append(l)
    return torch.cat(outs), torch.cat(lses)


def _mulhilo(m, x):
    """High and low word of the product of a 32-bit constant and 32-bit words held in int64."""
    lo, hi = m * (x & 0xFFFF), m * (x >> 16)
    mid = (lo >> 16) + (hi & 0xFFFF)
    return (hi >> 16) + (mid >> 16), ((mid & 0xFFFF) << 16) | (lo & 0xFFFF)


def _gumbel(seed, seq_id, step, V):
    """The sampler's noise [rows, V]: Philox4x32-10 with key = seed, counter = (v >> 2, step, sequence)."""
    blocks = (V + 3) // 4
    c0 = torch.arange(blocks, device="cuda")[None, :].expand(len(step), blocks)
    c1 = step.long()[:, None].expand_as(c0)
    c2, c3 = (seq_id & 0xFFFFFFFF)[:, None].expand_as(c0), (seq_id >> 32)[:, None].expand_as(c0)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c0)
        h1, l1 = _mulhilo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = (torch.stack([c0, c1, c2, c3], -1).reshape(len(step), 4 * blocks)[:, :V] >> 9).double().add_(0.5).mul_(2.0 ** -23)
    return u.log_().neg_().log_().neg_()


def _head(s, case, rows, pick):
    """Log-probs in blocks of rows; pick(z, r, n) names the tokens of rows r .. r + n."""
    w = s["weight"].double().t().contiguous()
    tokens, logps, lses = [], [], []
    for r in range(0, rows, 1024 if pick is None else 64):
        h = s["hidden"][r:r + (1024 if pick is None else 64)].double()
        z = torch.matmul(h, w).div_(case["T"])
        lse = torch.logsumexp(z, -1)
        tok = s["tokens"][r:r + len(h)].long() if pick is None else pick(z, r, len(h))
        tokens.append(tok.to(torch.int32))
        logps.append(z.gather(1, tok[:, None])[:, 0] - lse)
        lses.append(lse)
    return torch.cat(tokens), torch.cat(logps), torch.cat(lses)


def _sampled(s, case):
    def pick(z, r, n):
        return (z + _gumbel(s["seed"], s["seq_id"][r:r + n], s["step"][r:r + n], case["V"])).argmax(-1)
    return _head(s, case, case["C"], pick)


def _exact_batch(s, case):
    lens = torch.from_numpy(s["lens"].astype(np.int64)).cuda()
    b = len(lens)
    seq = torch.repeat_interleave(torch.arange(b, device="cuda"), lens)
    local = torch.arange(len(seq), device="cuda") - s["cu"].long()[seq]
    row = s["traj"].long()[seq]
    split = torch.minimum(s["boundary"][s["traj"].long(), 0], lens)
    earlier, old32 = local < split[seq], s["buf_logp"][row, local]
    cur, old, nan = s["logp_cur"].double(), old32.double(), torch.full_like(old32, math.nan)
    counted = s["mask"].bool() if s["mask"] is not None else torch.ones_like(earlier)
    r = (cur - old).exp()
    # the bounds and the advantage as the fp32 numbers that the call takes
    lo, hi = float(np.float32(1) - np.float32(0.2)), float(np.float32(1) + np.float32(0.28))
    rc, adv = r.clamp(lo, hi), s["adv"].double()[seq]
    t1, t2 = r * adv, rc * adv
    zero = torch.zeros_like(r)
    surr, grad = torch.where(counted, torch.minimum(t1, t2), zero), torch.where(counted & (t1 <= t2), t1, zero)
    per_seq = lambda x: torch.zeros(b, dtype=x.dtype, device="cuda").index_add_(0, seq, x)  # noqa: E731
    cnt, seq_surr = per_seq(counted.long()), per_seq(surr)
    means = torch.where(cnt > 0, seq_surr / cnt.clamp(min=1), torch.zeros_like(seq_surr))
    objective = torch.stack([seq_surr.sum() / cnt.sum().clamp(min=1), means.mean()])
    return {"tokens": s["buf_token"][row, local], "logp_buf": torch.where(earlier, old32, nan),
            "logp_roll": torch.where(earlier, nan, old32), "split": split.to(torch.int32),
            "ratio": torch.where(counted, r, zero), "clipped": torch.where(counted, rc, zero),
            "seq_sum": per_seq(torch.where(counted, rc, zero)), "seq_cnt": cnt.to(torch.int32),
            "seq_nclip": per_seq((counted & (rc != r)).long()).to(torch.int32), "surr": surr, "grad": grad,
            "seq_surr": seq_surr, "seq_cnt2": cnt.to(torch.int32), "objective": objective}


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "batch":
        return _exact_batch(s, case)
    if kind == "attn":
        out, lse = _paged_attn(s, case)
        return {"out": out, "lse": lse}
    if kind == "sample":
        token, logprob, lse = _sampled(s, case)
        return {"token": token, "logprob": logprob, "lse": lse}
    if kind == "given":
        _, logprob, lse = _head(s, case, case["M"], None)
        return {"logprob": logprob, "lse": lse}
    if kind == "prefill":
        outs, lses, at = [], [], 0
        for n in s["lens"].tolist():
            o, l = _softmax_attn(*(s[x][at:at + n].double() for x in "qkv"), 128 ** -0.5, True)
            outs.append(o)
            lses.append(l)
            at += n
        return {"out": torch.cat(outs), "lse": torch.cat(lses), "k_cache": None, "v_cache": None}
    last = s["ctx_len"].long() - 1
    page = s["block_table"][torch.arange(case["C"], device="cuda"), last // case["page"]].long()
    for name in ("k", "v"):
        s[name + "_cache"][page, :, last % case["page"]] = s[name + "_new"]
    out, lse = _paged_attn(s, case)
    token, logprob, lm_lse = _sampled(s, case)
    return {"out": out, "lse": lse, "token": token, "logprob": logprob, "lm_lse": lm_lse, "pool_seq": None, "pool_ctx": None,
            "pool_step": None, "k_cache": None, "v_cache": None, "buf_token": None, "buf_logp": None, "buf_tag": None}
