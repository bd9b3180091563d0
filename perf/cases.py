"""Workloads of the library: the calls a training or serving program makes, over the range of sizes it makes them at.

Kinds of call (`kind`):
  estimator  rapid_seq_logratio + rapid_group_advantage on stored log-probs (no LM head): logging and reward shaping
  logprob    rapid_logprob_fwd: log-probs of sampled tokens under the current or the behaviour policy
  step       rapid_iw_pg_loss_fwd_bwd: one mini-batch of the off-policy update, gradients of the hidden states and of W;
             with `optimizer` also the weight update that follows it in the inner loop
  clip       rapid_clip_pg_loss_fwd_bwd: the loss step of the GRPO and DAPO baselines
  adamw      rapid_adamw_step on an LM head's fp32 master weights, bf16 copy out

Sizes of a batch: `prompts` x `G` generations with lengths uniform in [len_lo, len_hi], padded to len_hi; LM head [d, V], stored
[d, V] (`layout` "dv") or, as checkpoints store it, [V, d] ("vd").  Inputs are those of paper_2510_03515_amd.workloads, with the
behaviour weights as close to the current ones as a few off-policy steps leave them (generation-level log ratios of order one).
"""
import math

import torch

from paper_2510_03515_amd import binding as rb
from paper_2510_03515_amd import workloads as wl

V_QWEN = 151936


def _batch(kind, name=None, **kw):
    c = dict(kind=kind, dtype="bf16", d=1536, V=V_QWEN, layout="dv", prompts=8, G=8, len_lo=64, len_hi=512)
    if kind == "step":
        c.update(cache=False, dw="f32", accumulate=False, rms=False, optimizer="none")
    if kind == "clip":
        c.update(cache=False, variant="grpo")
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # statistics of one tiny batch (the fp32 check case's 8 x 4 generations): two calls, nothing but launches
        dict(name="estimator_tiny", kind="estimator", prompts=8, G=4, len_lo=8, len_hi=32),
        # the fp32 check case: an update step on a toy head, where the number of launches is the time
        _batch("step", "step_f32_tiny", dtype="f32", d=64, V=1000, prompts=8, G=4, len_lo=8, len_hi=32),
        # the synthetic bandit's whole inference batch in fp32: the accuracy path on more than a toy
        _batch("step", "step_f32_bandit", dtype="f32", d=256, V=4096, prompts=64, G=8, len_lo=8, len_hi=48),
        # one inner step of the synthetic bandit in bf16: mini-batch step with the cache, then the SGD update of the head
        _batch("step", "inner_step_bandit", d=256, V=4096, prompts=8, G=8, len_lo=8, len_hi=48, cache=True, optimizer="sgd"),
        # a serving loop scores the tokens of a few sequences between decoding steps (1.5B-shaped head as checkpoints store it)
        _batch("logprob", "score_few", layout="vd", prompts=8, G=1, len_lo=8, len_hi=64),
        # behaviour log-probs of an inference batch, forward only (a quarter of the large forward-only workload)
        _batch("logprob", "score_batch", prompts=128, G=1, len_lo=1024, len_hi=1024),
        # per-device micro-batch of gradient accumulation: one prompt's 4 generations on a 1.5B-shaped head, default options
        _batch("step", "micro_step_accumulate", layout="vd", prompts=1, G=4, len_lo=64, len_hi=1024, accumulate=True),
        # GRPO baseline's step on an ordinary mini-batch, default options (logits regenerated in the backward), KL term on
        _batch("clip", "grpo_step", prompts=4, G=8, len_lo=64, len_hi=768),
        # 3B-shaped head with the model's final norm folded in, bf16 gradient for a bf16 optimiser, cached backward
        _batch("step", "step_3b_rmsnorm", layout="vd", d=2048, prompts=4, G=16, len_lo=64, len_hi=512, rms=True, dw="bf16", cache=True),
        # 0.5B-shaped mini-batch, cached backward
        _batch("step", "step_0.5b", d=896, prompts=16, G=8, len_lo=128, len_hi=1024, cache=True),
        # the headline workload: 1.5B-shaped mini-batch, cached backward in chunks of whole groups
        _batch("step", "step_1.5b", d=1536, prompts=32, G=8, len_lo=256, len_hi=2048, cache=True),
        # AdamW on the 0.5B-shaped head
        dict(name="adamw_0.5b", kind="adamw", d=896, V=V_QWEN),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _tokens(c):
    return c["prompts"] * c["G"] * (c["len_lo"] + c["len_hi"]) / 2


def draw(rng):
    kind = rng.choice(["estimator", "logprob", "logprob", "step", "step", "step", "clip", "f32", "adamw"])
    if kind == "adamw":
        return dict(kind=kind, d=8 * _log_int(rng, 8, 256), V=_log_int(rng, 1000, V_QWEN))
    while True:
        f32 = kind == "f32"
        hi = _log_int(rng, 16, 64 if f32 else 2048)
        sizes = dict(prompts=_log_int(rng, 1, 64), G=rng.choice([4, 6, 8, 16]), len_lo=max(1, int(hi * rng.uniform(0.05, 0.6))), len_hi=hi)
        if kind == "estimator":
            return dict(sizes, kind=kind)
        # hidden size a multiple of 8 in bf16 (any in fp32); vocabularies of toy heads up to the large one, odd ones among them
        sizes.update(d=_log_int(rng, 16, 256) if f32 else 8 * _log_int(rng, 8, 256), V=_log_int(rng, 500, 4096 if f32 else V_QWEN),
                     layout=rng.choice(["dv", "vd"]))
        if f32:
            c = _batch("step", dtype="f32", **sizes)
        elif kind == "logprob":
            c = _batch("logprob", **dict(sizes, G=1))
        elif kind == "clip":
            c = _batch("clip", cache=rng.random() < 0.5, variant=rng.choice(["grpo", "dapo"]), **sizes)
        else:
            dw = rng.choice(["f32", "f32", "bf16"])
            c = _batch("step", cache=rng.random() < 0.6, dw=dw, accumulate=dw == "f32" and rng.random() < 0.3,
                       rms=rng.random() < 0.3, optimizer="sgd" if dw == "f32" and rng.random() < 0.2 else "none", **sizes)
        top = 64 * 8 * 28 * 256 * 4096.0 if f32 else 32 * 8 * 1152 * 1536 * float(V_QWEN)
        # no more than the largest listed batch of its type, padding included; regenerating costs a third more
        if c["prompts"] * c["G"] * c["len_hi"] <= 32 * 8 * 2048 and _tokens(c) * c["d"] * c["V"] <= top * (1.0 if c.get("cache") else 0.75):
            return c


def _spec(case):
    fields = dict(d=case["d"], V=case["V"], prompts=case["prompts"], G=case["G"], len_lo=case["len_lo"], len_hi=case["len_hi"])
    spec = wl.WorkloadSpec("case", case["dtype"], sigma=0.01, reward="bernoulli", reward_p=0.4, **fields)
    return wl.calibrated(spec)


def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if kind == "estimator":
        N, T = case["prompts"] * case["G"], case["len_hi"]
        length = torch.randint(case["len_lo"], T + 1, (N, 1), generator=gen, device="cuda")
        mask = (torch.arange(T, device="cuda")[None, :] < length).to(torch.uint8)
        logp_b = -8.0 - 3.0 * torch.rand((N, T), generator=gen, device="cuda")
        logp = logp_b + math.sqrt(0.5 / T) * torch.randn((N, T), generator=gen, device="cuda")
        rewards = (torch.rand(N, generator=gen, device="cuda") < 0.4).float()
        group = (torch.arange(N, device="cuda") // case["G"]).to(torch.int32)
        return dict(kind=kind, logp=logp * mask, logp_b=logp_b * mask, mask=mask, rewards=rewards, group=group, K=case["prompts"])
    if kind == "adamw":
        shape = (case["d"], case["V"])
        s = dict(kind=kind, master=torch.randn(shape, generator=gen, device="cuda") * 0.02,
                 grad=torch.randn(shape, generator=gen, device="cuda") * 1e-3,
                 m=torch.randn(shape, generator=gen, device="cuda") * 1e-3,
                 v=torch.rand(shape, generator=gen, device="cuda") * 1e-6)
        return dict(s, w_out=torch.empty(shape, dtype=torch.bfloat16, device="cuda"), step=100)

    w = wl.make_workload(_spec(case), seed=seed, device="cuda")
    layout = rb.W_VD if case["layout"] == "vd" else rb.W_DV
    W = w["W"].t().contiguous() if case["layout"] == "vd" else w["W"]
    s = dict(kind=kind, case=case, hidden=w["hidden"], W=W, layout=layout, tokens=w["tokens"], mask=w["mask"])
    if kind == "logprob":
        nbytes = rb.rapid_workspace_bytes(rb.OP_LOGPROB_FWD, *w["hidden"].shape, case["V"], 1, rb.DTYPE_BF16)
        return dict(s, workspace=rb.alloc_workspace(nbytes))
    rms = {}
    if case.get("rms"):
        rms = dict(rms_weight=(1.0 + 0.1 * torch.randn(case["d"], generator=gen, device="cuda")).to(torch.bfloat16))
    logp_b, _ = rb.rapid_logprob_fwd(w["hidden"], w["W_old"], w["tokens"], w["mask"], **rms)
    max_tokens = int(w["mask"].sum().item()) if case["cache"] else 0
    dw_dtype = torch.bfloat16 if case.get("dw") == "bf16" else torch.float32
    buffers = rb.IwPgBuffers(w["hidden"], W, w["K"], layout, dw_dtype=dw_dtype, logits_cache=case["cache"])
    buffers.dW.zero_()
    s.update(logp_b=logp_b, rewards=w["rewards"], group=w["group_ids"], K=w["K"], buffers=buffers, max_tokens=max_tokens, rms=rms)
    if kind == "clip":      # the reference policy: another copy of the head, as far away as the behaviour policy
        noise = torch.randn(logp_b.shape, generator=gen, device="cuda")
        s["logp_ref"] = logp_b + math.sqrt(0.5 / logp_b.shape[1]) * noise * w["mask"]
    elif case["optimizer"] == "sgd":
        s["master"] = W.float()
    return s


def run(s):
    if s["kind"] == "estimator":
        seq, tok = rb.rapid_seq_logratio(s["logp"], s["logp_b"], s["mask"], want_tokens=True)
        return dict(rb.rapid_group_advantage(s["rewards"], s["group"], s["K"], seq_logratio=seq), seq=seq, tok=tok)
    if s["kind"] == "adamw":
        rb.rapid_adamw_step(s["master"], s["grad"], s["m"], s["v"], s["step"], 1e-6, weight_decay=0.01, w_out=s["w_out"])
        return dict(master=s["master"], m=s["m"], v=s["v"], w=s["w_out"])
    if s["kind"] == "logprob":
        logp, lse = rb.rapid_logprob_fwd(s["hidden"], s["W"], s["tokens"], s["mask"], w_layout=s["layout"], want_lse=True,
                                         workspace=s["workspace"])
        return dict(logp=logp, lse=lse)
    case = s["case"]
    common = dict(buffers=s["buffers"], w_layout=s["layout"], logits_cache=case["cache"], max_tokens=s["max_tokens"])
    if s["kind"] == "clip":
        ref = s["logp_ref"] if case["variant"] == "grpo" else None
        out = rb.rapid_clip_pg_loss_fwd_bwd(s["hidden"], s["W"], s["tokens"], s["mask"], s["logp_b"], ref, s["rewards"],
                                            s["group"], s["K"], variant=case["variant"], **common)
        return dict(loss=out.loss, dhidden=out.dhidden, dW=out.dW, logp=out.logp_cur, adv=out.adv)
    out = rb.rapid_iw_pg_loss_fwd_bwd(s["hidden"], s["W"], s["tokens"], s["mask"], s["logp_b"], s["rewards"], s["group"],
                                      s["K"], accumulate_dw=case["accumulate"], **common, **s["rms"])
    got = dict(loss=out.loss, dhidden=out.dhidden, dW=out.dW, logp=out.logp_cur, seq=out.seq_logratio, adv=out.adv)
    if case["rms"]:
        got["drms"] = out.drms_weight
    if case["optimizer"] == "sgd":
        rb.rapid_sgd_step(s["master"], out.dW, 1e-6, w_out=s["W"])
        got.update(master=s["master"], W=s["W"])
    return got


def work(case):
    if case["kind"] == "adamw":     # gradient, weights and two moments in; weights, moments and the bf16 copy out
        n = case["d"] * case["V"]
        return dict(bytes=30 * n, flops=15 * n)
    N, T, M = case["prompts"] * case["G"], case["len_hi"], _tokens(case)
    if case["kind"] == "estimator":
        return dict(bytes=N * T * 13 + N * 24, flops=3 * N * T)
    e, d, V = (4 if case["dtype"] == "f32" else 2), case["d"], case["V"]
    if case["kind"] == "logprob":   # valid hidden rows, W and tokens in; log-prob and log-sum-exp out
        return dict(bytes=M * d * e + d * V * e + N * T * 13, flops=2 * M * d * V)
    # Gradients: the rows of a group whose rewards are all 0 are known to be zero (not under a KL term)
    live = 1.0 if case["kind"] == "clip" and case["variant"] == "grpo" else 1.0 - 0.6 ** case["G"]
    b = M * d * e + N * T * d * e + d * V * e + N * T * 21
    b += d * V * (2 if case.get("dw") == "bf16" else 8 if case.get("accumulate") else 4)
    b += d * V * 14 if case.get("optimizer") == "sgd" else 0
    return dict(bytes=b, flops=(2 + 4 * live) * M * d * V)


def tolerance(case):
    # About four times the largest difference seen from the same results formed in 64 bits.
    if case["kind"] == "adamw":      # the bf16 copy: an fp32 rounding turns about one element in 10^5 into its neighbour
        return {"rel": 6e-5, "max": 0.01}
    if case["kind"] == "estimator":  # sums in 64 bits, results in fp32
        return {"rel": 2e-7}
    if case["kind"] == "logprob":
        return {"rel": 1e-7}
    # A generation's coefficient is exp(sum of its fp32 log-prob differences).  `max`: an element of dW is a sum over tokens
    # whose terms can be far larger than the root mean square of dW
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 0.99}
