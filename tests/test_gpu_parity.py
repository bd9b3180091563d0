"""Parity of the HIP path (through the C ABI) against the float64 oracle, element by element, on
seeded synthetic inputs small enough for the oracle to finish in seconds but spanning several
tiles and ragged tails.  Tolerances: integer/index outputs bit-exact; loss rel <= 1e-3;
dHidden/dW relative (Frobenius) error <= 2e-2 in bf16 and <= 1e-5 in fp32, and every single
element of both within 3 * 2^-8 (bf16; 1e-5 fp32) of the largest magnitude in its token row (dHidden) or
vocabulary column (dW) of the oracle's tensor (parity_bounds.py)."""
import math

import numpy as np
import pytest
import torch

import parity_bounds as pb
from oracle import rapid_oracle as orc
from paper_2510_03515_amd import workloads as wl

pytestmark = pytest.mark.gpu

LOSS_RTOL = 1e-3
GRAD_RTOL = {"bf16": 2e-2, "f32": 1e-5}
LOGP_ATOL = {"bf16": 2e-5, "f32": 2e-6}     # |logp| ~ 7..12, fp32 storage: a few ulp
S_ATOL = 1e-3


@pytest.fixture(scope="module")
def rb():
    from paper_2510_03515_amd import binding
    binding.load()
    assert torch.cuda.is_available()
    return binding


def _np(t):
    return t.detach().float().cpu().numpy().astype(np.float64) if t.is_floating_point() else t.cpu().numpy()


def _rel(a, ref):
    a, ref = np.asarray(a, np.float64), np.asarray(ref, np.float64)
    return float(np.linalg.norm(a - ref) / max(np.linalg.norm(ref), 1e-300))


def _dh_ok(got, ref, dtype="bf16", rel=None, slack=None):
    """dHidden against the oracle: Frobenius norm, and every element within its row's bound (slack: what
    each generation's coefficient may be off by because stored log-probs are floats, parity_bounds.py)."""
    got = _np(got) if torch.is_tensor(got) else got
    assert _rel(got, ref) <= GRAD_RTOL[dtype]
    rel = pb.REL[dtype] if rel is None else rel
    pb.assert_dhidden_close(got, ref, dtype, rel if slack is None else rel + slack[:, None, None])


def _dw_ok(got, ref, dtype="bf16", rel=None, slack=None):
    """dW ([d, V]) against the oracle: Frobenius norm, and every element within its column's bound (a
    column mixes the generations: the largest slack among them)."""
    got = _np(got) if torch.is_tensor(got) else got
    assert _rel(got, ref) <= GRAD_RTOL[dtype]
    rel = pb.REL[dtype] if rel is None else rel
    pb.assert_dw_close(got, ref, dtype, rel if slack is None else rel + float(slack.max()))


def _make(spec, seed=0):
    w = wl.make_workload(spec, seed=seed, device="cpu")
    g = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in w.items()}
    return w, g


def _oracle_inputs(w):
    return (_np(w["hidden"]), _np(w["W"]), _np(w["tokens"]), _np(w["mask"]))


# ----------------------------------------------------------------------------- integer work
@pytest.mark.parametrize("N,T,p", [(1, 1, 1.0), (5, 9, 0.6), (37, 200, 0.5), (3, 1500, 0.9), (64, 64, 0.0), (20011, 3, 0.6)])
def test_compaction_bit_exact(rb, N, T, p):
    print(f"compaction N={N} T={T} p={p}", flush=True)
    rng = np.random.default_rng(N * 1000 + T)
    mask = (rng.random((N, T)) < p).astype(np.uint8)      # arbitrary pattern, not only right padding
    seq_len, cu, row_index = rb.rapid_compaction(torch.from_numpy(mask).cuda())
    torch.cuda.synchronize()
    o_len, o_cu, o_rows = orc.compaction(mask)
    assert np.array_equal(seq_len.cpu().numpy(), o_len)
    assert np.array_equal(cu.cpu().numpy(), o_cu)
    M = int(o_cu[-1])
    assert np.array_equal(row_index.cpu().numpy()[:M], o_rows)


@pytest.mark.parametrize("mode", ["eq2", "eq5", "eq4", "loo1", "loo2"])
def test_group_advantage(rb, mode):
    print(f"group_advantage {mode}", flush=True)
    rng = np.random.default_rng(3)
    N, K = 1000, 37
    R = rng.random(N).astype(np.float32)
    gid = rng.integers(0, K - 2, size=N).astype(np.int32)     # ragged, shuffled, two empty groups
    s = (rng.normal(size=N) * 0.8).astype(np.float32)
    kw = dict(eq2=dict(s=None), eq5=dict(s=s, eta=2.0), eq4=dict(s=s, eta=math.inf),
              loo1=dict(s=s, eta=2.0, baseline_mode=1), loo2=dict(s=s, eta=2.0, baseline_mode=2))[mode]
    ref = orc.group_advantage(R, gid, K, **kw)
    out = rb.rapid_group_advantage(torch.from_numpy(R).cuda(), torch.from_numpy(gid).cuda(), K,
                                   seq_logratio=None if kw["s"] is None else torch.from_numpy(s).cuda(),
                                   eta=kw.get("eta", 2.0), baseline_mode=kw.get("baseline_mode", 0))
    torch.cuda.synchronize()
    assert np.array_equal(out["group_size"].cpu().numpy(), ref["group_size"])     # bit-exact
    assert np.allclose(_np(out["adv"]), ref["adv"], atol=2e-6)
    assert np.allclose(_np(out["weight"]), ref["weight"], rtol=1e-6)
    assert np.allclose(_np(out["group_mean"]), ref["group_mean"], atol=1e-6)
    assert np.allclose(_np(out["group_std"]), ref["group_std"], atol=1e-6)


def test_group_advantage_hand_example_and_status(rb):
    rho = torch.tensor([4.0, 1.0, 1.0, 0.5]).log().cuda()
    R = torch.tensor([1.0, 0.0, 0.0, 1.0]).cuda()
    gid = torch.zeros(4, dtype=torch.int32).cuda()
    out = rb.rapid_group_advantage(R, gid, 1, seq_logratio=rho, eta=2.0)
    assert np.allclose(_np(out["adv"]), [0.375, -0.625, -0.625, 0.375], atol=1e-6)
    status = torch.zeros(1, dtype=torch.int32).cuda()
    bad_gid = torch.tensor([0, 5, -1, 0], dtype=torch.int32).cuda()
    out = rb.rapid_group_advantage(R, bad_gid, 1, dev_status=status)
    torch.cuda.synchronize()
    assert status.item() & rb.STATUS_BAD_GROUP
    assert out["group_size"].item() == 2 and _np(out["adv"])[1] == 0.0


# ----------------------------------------------------------------------------- log-probabilities
SPECS = {
    "f32_cfg0": wl.CONFIGS[0],
    "f32_ragged": wl.small_spec("f32_ragged", "f32", d=50, V=777, prompts=3, G=3, len_lo=1, len_hi=70),
    "bf16_small": wl.small_spec("bf16_small", "bf16", d=128, V=1000, prompts=4, G=4, len_lo=3, len_hi=40),
    "bf16_ragged": wl.small_spec("bf16_ragged", "bf16", d=200, V=1321, prompts=5, G=3, len_lo=1, len_hi=90,
                                 sigma=0.02, reward="uniform"),
}


@pytest.mark.parametrize("name", list(SPECS))
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_logprob_fwd(rb, name, layout):
    print(f"logprob_fwd {name} {layout}", flush=True)
    spec = SPECS[name]
    w, g = _make(spec)
    H, W, tok, mask = _oracle_inputs(w)
    ref_lp, ref_lse = orc.logprob(H, W, tok, mask)
    Wg = g["W"] if layout == "dv" else g["W"].t().contiguous()
    lp, lse = rb.rapid_logprob_fwd(g["hidden"], Wg, g["tokens"], g["mask"],
                                   w_layout=rb.W_DV if layout == "dv" else rb.W_VD, want_lse=True)
    torch.cuda.synchronize()
    assert np.abs(_np(lp) - ref_lp).max() <= LOGP_ATOL[spec.dtype]
    assert np.abs(_np(lse) - ref_lse).max() <= LOGP_ATOL[spec.dtype]
    assert np.all(_np(lp)[mask == 0] == 0.0)


def test_logprob_closed_form_and_temperature(rb):
    spec = SPECS["bf16_small"]
    w, g = _make(spec)
    lp, lse = rb.rapid_logprob_fwd(g["hidden"], torch.zeros_like(g["W"]), g["tokens"], g["mask"], want_lse=True)
    torch.cuda.synchronize()
    m = _np(g["mask"]) != 0
    assert np.allclose(_np(lp)[m], -math.log(spec.V), atol=2e-6)       # W = 0 -> uniform over V
    assert np.allclose(_np(lse)[m], math.log(spec.V), atol=2e-6)
    H, W, tok, mask = _oracle_inputs(w)
    ref, _ = orc.logprob(H, W, tok, mask, temperature=0.7)
    lp, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"], temperature=0.7)
    assert np.abs(_np(lp) - ref).max() <= LOGP_ATOL["bf16"]


# ----------------------------------------------------------------------------- fused forward + backward
def _run_pair(rb, spec, seed=0, layout="dv", min_ws=False, dw_dtype=torch.float32, **kw):
    w, g = _make(spec, seed)
    H, W, tok, mask = _oracle_inputs(w)
    lay = rb.W_DV if layout == "dv" else rb.W_VD
    Wg = g["W"] if layout == "dv" else g["W"].t().contiguous()
    Wold = g["W_old"] if layout == "dv" else g["W_old"].t().contiguous()
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], Wold, g["tokens"], g["mask"], w_layout=lay,
                                     temperature=kw.get("temperature", 1.0))
    buf = rb.IwPgBuffers(g["hidden"], Wg, w["K"], w_layout=lay, dw_dtype=dw_dtype, minimum_workspace=min_ws,
                         logits_cache=kw.get("logits_cache", False))
    coef = kw.pop("coef_override", None)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], Wg, g["tokens"], g["mask"], logp_b, g["rewards"],
                                      g["group_ids"], w["K"], buffers=buf, w_layout=lay,
                                      coef_override=None if coef is None else torch.from_numpy(coef).cuda(), **kw)
    torch.cuda.synchronize()
    okw = {k: v for k, v in kw.items() if k not in ("accumulate_dw", "logits_cache")}   # the rest means the same to the oracle
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"],
                                 coef_override=coef, **okw)
    # what the float storage of the log-probs may do to each generation's coefficient (none if they are given)
    ref["slack"] = None if coef is not None else pb.coefficient_slack(ref, _np(w["rewards"]), mask)
    return w, out, ref


def _check_pair(rb, spec, out, ref, layout="dv"):
    dW = _np(out.dW) if layout == "dv" else _np(out.dW).T
    assert out.dev_status.item() == 0
    assert np.abs(_np(out.seq_logratio) - ref["seq_logratio"]).max() <= S_ATOL
    assert np.abs(_np(out.logp_cur) - ref["logp_cur"]).max() <= LOGP_ATOL[spec.dtype]
    assert np.abs(_np(out.tok_logratio) - ref["tok_logratio"]).max() <= 2 * LOGP_ATOL[spec.dtype]
    assert np.allclose(_np(out.adv), ref["adv"], atol=1e-3 if spec.dtype == "bf16" else 1e-5)
    loss = out.loss.item()
    # The loss is a sum of per-generation terms that may cancel (on-policy, complete groups: exactly 0 in the
    # library, whose ratios are exactly 1 there, and a rounding residue in the oracle, whose current log-probs
    # are float64 against float stored ones): each term gets the slack its coefficient has.
    tol = LOSS_RTOL * max(abs(ref["loss"]), 1e-30)
    if ref.get("slack") is not None:
        per_gen = np.abs(np.asarray(ref["g"], np.float64)).reshape(len(ref["adv"]), -1).max(axis=1)
        tol += float((per_gen * np.maximum(ref["slack"], 2.0 ** -23)).sum())
    assert abs(loss - ref["loss"]) <= tol, (loss, ref["loss"], tol)
    _dh_ok(out.dhidden, ref["dH"], spec.dtype, slack=ref.get("slack"))
    _dw_ok(dW, ref["dW"], spec.dtype, slack=ref.get("slack"))
    mask0 = ref["logp_cur"] == 0
    assert np.all(_np(out.dhidden)[mask0 & (np.abs(ref["dH"]).sum(-1) == 0)] == 0.0)
    dg = out.read_diag()
    assert dg["n_tokens"] == ref["n_tokens"]                     # bit-exact
    assert dg["n_sequences"] == len(ref["adv"])
    near = int((np.abs(ref["seq_logratio"] - math.log(2.0)) < 1e-3).sum())
    assert abs(dg["n_clipped"] - ref["n_clipped"]) <= near
    assert abs(dg["mean_log_w"] - ref["mean_log_w"]) <= 1e-3
    assert abs(dg["mean_abs_log_w"] - ref["mean_abs_log_w"]) <= 1e-3


@pytest.mark.parametrize("name", list(SPECS))
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_fwd_bwd_parity(rb, name, layout):
    print(f"fwd_bwd {name} {layout}", flush=True)
    spec = SPECS[name]
    w, out, ref = _run_pair(rb, spec, layout=layout)
    _check_pair(rb, spec, out, ref, layout)


@pytest.mark.parametrize("name", ["f32_ragged", "bf16_ragged"])
def test_fwd_bwd_minimum_workspace(rb, name):
    """Smallest workspace: the backward runs in 256-row chunks (several chunks, ragged last one)."""
    print(f"fwd_bwd min workspace {name}", flush=True)
    spec = SPECS[name]
    w, out, ref = _run_pair(rb, spec, min_ws=True)
    _check_pair(rb, spec, out, ref)


@pytest.mark.parametrize("name", ["f32_cfg0", "bf16_small"])
def test_fwd_bwd_options(rb, name):
    print(f"fwd_bwd options {name}", flush=True)
    spec = SPECS[name]
    for kw in (dict(coef_mode=1), dict(baseline_mode=1), dict(baseline_mode=2), dict(eta=math.inf),
               dict(loss_scale=0.25), dict(temperature=0.8), dict(normalized_grads=True), dict(eta=1.05)):
        print("  ", kw, flush=True)
        w, out, ref = _run_pair(rb, spec, **kw)
        _check_pair(rb, spec, out, ref)
        if kw.get("normalized_grads"):
            assert abs(out.read_diag()["grad_log_scale"] - ref["grad_log_scale"]) <= 1e-3


def test_cross_entropy_special_case(rb):
    """coef_override g = -1/M: mean token cross-entropy of a linear layer (heavy kernels checked
    independently of the RL scalars)."""
    spec = SPECS["bf16_small"]
    w0 = wl.make_workload(spec, seed=0, device="cpu")
    M = int(w0["mask"].sum())
    coef = np.full(spec.N, -1.0 / M, np.float32)
    w, out, ref = _run_pair(rb, spec, coef_override=coef)
    _dh_ok(out.dhidden, ref["dH"])
    _dw_ok(out.dW, ref["dW"])
    assert abs(out.loss.item() - coef.astype(np.float64).sum()) <= 1e-5
    assert np.abs(_np(out.dW).sum(axis=1)).max() <= 1e-3 * np.abs(_np(out.dW)).sum(axis=1).max()


def test_dw_bf16_and_accumulate(rb):
    spec = SPECS["bf16_small"]
    w, out, ref = _run_pair(rb, spec, dw_dtype=torch.bfloat16)
    assert out.dW.dtype == torch.bfloat16
    _dw_ok(out.dW, ref["dW"], rel=2.0 ** -6)            # the stored gradient is rounded once more
    # accumulate: dW_out starts at a known value
    w, g = _make(spec)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"])
    buf.dW.fill_(0.5)
    rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"],
                                g["group_ids"], w["K"], buffers=buf, accumulate_dw=True)
    torch.cuda.synchronize()
    assert _rel(_np(buf.dW) - 0.5, ref["dW"]) <= GRAD_RTOL["bf16"]
    # element by element, up to the fp32 rounding of 0.5 + x (half an ulp of 0.5 = 3e-8)
    err = np.abs(_np(buf.dW) - 0.5 - ref["dW"])
    assert np.all(err <= 3 * 2.0 ** -8 * np.abs(ref["dW"]).max(axis=0, keepdims=True) + 6e-8)


@pytest.mark.parametrize("name", ["f32_cfg0", "bf16_small"])
def test_on_policy_reduction_exact(rb, name):
    """Behaviour log-probs produced by the library itself with the same W: every generation-level
    log ratio is exactly 0, every weight exactly 1, advantages equal Eq. (2) and the loss is 0."""
    spec = SPECS[name]
    w, g = _make(spec)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"],
                                      g["group_ids"], w["K"])
    torch.cuda.synchronize()
    assert torch.equal(out.logp_cur, logp_b)                                   # bitwise
    assert torch.all(out.seq_logratio == 0) and torch.all(out.tok_logratio == 0)
    on = orc.group_advantage(_np(w["rewards"]), _np(w["group_ids"]), w["K"], s=None)
    assert np.allclose(_np(out.adv), on["adv"], atol=1e-6)
    assert abs(out.loss.item()) <= 1e-7
    dg = out.read_diag()
    assert dg["n_clipped"] == 0 and dg["mean_log_w"] == 0.0
    # and twice the same call gives bitwise identical gradients (no atomics, fixed order)
    out2 = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"],
                                       g["group_ids"], w["K"])
    torch.cuda.synchronize()
    assert torch.equal(out.dW, out2.dW) and torch.equal(out.dhidden, out2.dhidden)
    # no behaviour log-probs at all = the on-policy estimator of Sec. 3.3: the same bits
    out3 = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], None, g["rewards"],
                                       g["group_ids"], w["K"])
    torch.cuda.synchronize()
    for k in ("loss", "dW", "dhidden", "adv", "seq_logratio", "logp_cur"):
        assert torch.equal(getattr(out3, k), getattr(out, k)), k


def test_edge_cases(rb):
    spec = SPECS["bf16_small"]
    w, g = _make(spec)
    # (a) one generation with no valid token, (b) everything masked
    mask = g["mask"].clone()
    mask[2] = 0
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], mask)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], mask, logp_b, g["rewards"],
                                      g["group_ids"], w["K"])
    torch.cuda.synchronize()
    H, W, tok, _ = _oracle_inputs(w)
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, _np(mask), _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"])
    assert out.seq_logratio[2].item() == 0.0 and torch.all(out.dhidden[2] == 0)
    _dw_ok(out.dW, ref["dW"])
    _dh_ok(out.dhidden, ref["dH"])
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    mask.zero_()
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], mask)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], mask, logp_b, g["rewards"],
                                      g["group_ids"], w["K"])
    torch.cuda.synchronize()
    assert torch.all(logp_b == 0) and torch.all(out.dW == 0) and torch.all(out.dhidden == 0)
    assert out.read_diag()["n_tokens"] == 0
    # (c) token id outside the vocabulary at an unmasked position: flagged, no fault
    tok = g["tokens"].clone()
    tok[0, 0] = spec.V + 5
    status = torch.zeros(1, dtype=torch.int32).cuda()
    rb.rapid_logprob_fwd(g["hidden"], g["W"], tok, g["mask"], dev_status=status)
    torch.cuda.synchronize()
    assert status.item() & rb.STATUS_BAD_TOKEN


@pytest.mark.parametrize("shape", [dict(d=8, V=5, prompts=1, G=2, len_lo=1, len_hi=1),
                                   dict(d=24, V=300, prompts=2, G=2, len_lo=1, len_hi=3),
                                   dict(d=264, V=257, prompts=3, G=2, len_lo=100, len_hi=130)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_smallest_and_off_tile_shapes(rb, shape, dtype):
    """The smallest accepted shapes (one token per generation, d = 8, a vocabulary of 5; two generations,
    because a group of one has the advantage R (1 - w), a difference of nearly equal numbers whose
    fp32 rounding no gradient tolerance survives) and sizes just past a tile
    boundary (d = 256 + 8, V = 256 + 1, more than 256 rows), in both backward modes, with the
    token-level weight as well; and a batch without a single valid token in the cache mode."""
    print(f"small shapes {shape} {dtype}", flush=True)
    spec = wl.small_spec("edge", dtype, reward="uniform", **shape)
    for kw in (dict(), dict(logits_cache=True), dict(logits_cache=True, ratio_level=1, coef_mode=1)):
        if kw.get("logits_cache") and dtype != "bf16":
            continue
        w, out, ref = _run_pair(rb, spec, **kw)
        _check_pair(rb, spec, out, ref)
    if dtype == "bf16":
        w, g = _make(spec)
        mask = torch.zeros_like(g["mask"])
        wgt = torch.ones(spec.d, dtype=torch.bfloat16, device="cuda")
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], mask, None, g["rewards"], g["group_ids"], w["K"],
                                          logits_cache=True, rms_weight=wgt)
        torch.cuda.synchronize()
        assert out.dev_status.item() == 0 and out.read_diag()["n_tokens"] == 0
        assert torch.all(out.dW == 0) and torch.all(out.dhidden == 0) and torch.all(out.drms_weight == 0)
        assert torch.all(out.logp_cur == 0) and torch.all(out.seq_logratio == 0)


def test_seeded_random_shapes_and_options(rb):
    """Twelve seeded draws of shape (d a multiple of 8 up to 400, V up to 2000, up to ~1500 token rows)
    and options (layout, backward mode, coefficient mode, ratio level, baseline, temperature, dW
    dtype), each against the oracle element by element.  (Behaviour weights always differ from the
    current ones here: on-policy the loss is an exact zero, which has its own test.)"""
    rng = np.random.default_rng(2024)
    for case in range(12):
        d = int(rng.integers(1, 51)) * 8
        V = int(rng.integers(2, 2001))
        prompts, G = int(rng.integers(1, 6)), int(rng.integers(2, 5))
        hi = int(rng.integers(1, 120))
        lo = int(rng.integers(1, hi + 1))
        spec = wl.small_spec(f"rand{case}", "bf16", d=d, V=V, prompts=prompts, G=G, len_lo=lo, len_hi=hi,
                             sigma=float(rng.choice([0.002, 0.005, 0.02])), reward=str(rng.choice(["bernoulli", "uniform"])))
        kw = dict(logits_cache=bool(rng.integers(0, 2)), coef_mode=int(rng.integers(0, 2)),
                  ratio_level=int(rng.integers(0, 2)), baseline_mode=int(rng.integers(0, 3)),
                  temperature=float(rng.choice([1.0, 0.7, 1.3])), normalized_grads=bool(rng.integers(0, 2)))
        layout = str(rng.choice(["dv", "vd"]))
        dw_dtype = torch.bfloat16 if rng.integers(0, 4) == 0 else torch.float32
        print(f"random case {case}: d={d} V={V} N={prompts * G} T={hi} {layout} {kw} dW={dw_dtype}", flush=True)
        w, out, ref = _run_pair(rb, spec, seed=case, layout=layout, dw_dtype=dw_dtype, **kw)
        if dw_dtype == torch.bfloat16:          # the stored gradient is itself rounded: compare apart from that
            dW = _np(out.dW) if layout == "dv" else _np(out.dW).T
            _dw_ok(dW, ref["dW"], rel=2.0 ** -6)
            out.dW = torch.from_numpy(ref["dW"] if layout == "dv" else ref["dW"].T.copy()).float().cuda()
        _check_pair(rb, spec, out, ref, layout)


def test_mfma_probe_and_forward_row_blocks(rb):
    """The probe reports a rate between zero and the published peak, random operands never beat
    integer ones by more than noise; the forward gives the same bits for any row-block size."""
    tf_int, ms = rb.rapid_mfma_probe(0, 20000)
    tf_rnd, _ = rb.rapid_mfma_probe(1, 20000)
    assert ms > 0 and 100.0 < tf_int < 2500.0 * 1.05
    assert 100.0 < tf_rnd < tf_int * 1.1
    spec = wl.small_spec("row_blocks", d=192, V=1500, prompts=6, G=4, len_lo=20, len_hi=90)
    w = wl.make_workload(spec, seed=3, device="cuda")
    ref, _ = rb.rapid_logprob_fwd(w["hidden"], w["W"], w["tokens"], w["mask"])
    try:
        rb.rapid_set_tuning(13, 1)   # one 256-row tile per launch: several launches, the last ones empty
        got, _ = rb.rapid_logprob_fwd(w["hidden"], w["W"], w["tokens"], w["mask"])
    finally:
        rb.rapid_set_tuning(13, 64)
    assert torch.equal(ref, got)


@pytest.mark.parametrize("name", ["bf16_small", "bf16_ragged"])
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_fwd_bwd_logits_cache(rb, name, layout):
    """logits_cache = 1: the forward keeps the bf16 ratios p_v / p_y, the backward contracts them instead
    of recomputing the logits; same tolerances against the oracle, same forward bits as the default mode."""
    print(f"fwd_bwd logits_cache {name} {layout}", flush=True)
    spec = SPECS[name]
    w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=True)
    _check_pair(rb, spec, out, ref, layout)
    w2, out2, _ = _run_pair(rb, spec, layout=layout)
    assert torch.equal(out.logp_cur, out2.logp_cur) and torch.equal(out.loss, out2.loss)
    for kw in (dict(temperature=0.8), dict(normalized_grads=True), dict(coef_mode=1, eta=1.05)):
        w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=True, **kw)
        _check_pair(rb, spec, out, ref, layout)


@pytest.mark.parametrize("name", ["f32_ragged", "bf16_small", "bf16_ragged"])
@pytest.mark.parametrize("cache", [False, True])
def test_fwd_bwd_token_level_ratio(rb, name, cache):
    """ratio_level 1 (every token carries its own ratio; not an estimator of the paper): every
    element against the oracle's token_coefficients path, both coefficient modes, plain and
    normalised, in both backward modes; on-policy it gives the generation-level gradients."""
    spec = SPECS[name]
    if cache and spec.dtype != "bf16":
        pytest.skip("the cache is a bf16 mode")
    print(f"fwd_bwd token-level {name} cache={cache}", flush=True)
    for kw in (dict(), dict(coef_mode=1, eta=1.05), dict(normalized_grads=True), dict(temperature=0.8, loss_scale=0.5)):
        w, out, ref = _run_pair(rb, spec, ratio_level=1, logits_cache=cache, **kw)
        _check_pair(rb, spec, out, ref)
        if kw.get("normalized_grads"):
            assert abs(out.read_diag()["grad_log_scale"] - ref["grad_log_scale"]) <= 1e-3
    w, g = _make(spec)
    lp, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    a = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lp, g["rewards"], g["group_ids"], w["K"],
                                    logits_cache=cache)
    b = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lp, g["rewards"], g["group_ids"], w["K"],
                                    logits_cache=cache, ratio_level=1)
    torch.cuda.synchronize()
    assert torch.equal(a.dhidden, b.dhidden) and torch.equal(a.dW, b.dW)      # all ratios exactly 1


@pytest.mark.parametrize("name", ["bf16_small", "bf16_ragged"])
@pytest.mark.parametrize("cache", [False, True])
def test_fwd_bwd_with_final_rmsnorm(rb, name, cache):
    """rms_weight: hidden is the input x of the final RMSNorm, applied while the rows are packed.
    The normalised state of a bf16 model is a bf16 tensor: the oracle normalises in float64 and rounds
    to bf16 (round_normed_hidden), the kernel forms the same product in fp64 and rounds once, so both
    take every rounding decision from the same value and the usual tolerances hold: log-probs, ratios,
    loss, dW, dL/dx and dL/dweight, every element."""
    print(f"fwd_bwd rmsnorm {name} cache={cache}", flush=True)
    spec = SPECS[name]
    w, g = _make(spec)
    rng = np.random.default_rng(31)
    d = spec.d
    x = (g["hidden"].float() * torch.from_numpy(rng.uniform(0.3, 3.0, size=g["hidden"].shape[:2] + (1,))).float().cuda()
         ).to(torch.bfloat16)                                         # rows of different scale: the norm matters
    wgt = torch.from_numpy(1.0 + 0.2 * rng.normal(size=d)).float().cuda().to(torch.bfloat16)
    eps = float(np.float32(1e-5))          # the ABI takes a float: give the oracle the same number
    logp_b, _ = rb.rapid_logprob_fwd(x, g["W_old"], g["tokens"], g["mask"], rms_weight=wgt, rms_eps=eps)
    out = rb.rapid_iw_pg_loss_fwd_bwd(x, g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], w["K"],
                                      logits_cache=cache, rms_weight=wgt, rms_eps=eps)
    lp2, _ = rb.rapid_logprob_fwd(x, g["W"], g["tokens"], g["mask"], rms_weight=wgt, rms_eps=eps)
    torch.cuda.synchronize()
    assert out.dev_status.item() == 0 and torch.equal(lp2, out.logp_cur)
    _, W, tok, mask = _oracle_inputs(w)
    ref = orc.iw_pg_loss_fwd_bwd(_np(x), W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"],
                                 rms_weight=_np(wgt), rms_eps=eps, round_normed_hidden=True)
    assert np.abs(_np(out.logp_cur) - ref["logp_cur"]).max() <= LOGP_ATOL["bf16"]
    assert np.abs(_np(out.seq_logratio) - ref["seq_logratio"]).max() <= S_ATOL
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dw_ok(out.dW, ref["dW"])
    _dh_ok(out.dhidden, ref["dH"], rel=2.0 ** -6)        # dL/dx: dL/dh was stored in bf16, then pushed through the norm
    assert _rel(_np(out.drms_weight), ref["d_rms_weight"]) <= GRAD_RTOL["bf16"]
    assert np.abs(_np(out.drms_weight) - ref["d_rms_weight"]).max() <= 2.0 ** -6 * np.abs(ref["d_rms_weight"]).max()
    assert np.all(_np(out.dhidden)[mask == 0] == 0.0)
    # the norm really is inside: unit weight and rows already of unit mean square change nothing but rounding
    ones = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    lp_plain, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    lp_unit, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"], rms_weight=ones, rms_eps=0.0)
    assert (lp_plain - lp_unit).abs().max().item() < 0.05 and not torch.equal(logp_b, lp_plain)


@pytest.mark.parametrize("scale", [25.0, 250.0])
def test_logits_cache_unlikely_sampled_tokens(rb, scale):
    """The cached values are relative to a reference known before the sweep: the sampled token's
    logit minus its behaviour log-prob (the behaviour policy's log-sum-exp, up to the token's drift).
    Peaked rows (logit spread ~7 and ~70) with tokens drawn uniformly put the sampled token 20..45
    and ~200 nats below the row maximum: with behaviour log-probs both stay inside the cache's range
    and meet the usual tolerances.  Without them (on-policy call) the reference is the sampled
    token's logit: the second case is then out of range, is reported through
    RAPID_STATUS_LOGIT_RANGE, and keeps exact log-probs and finite gradients."""
    print(f"logits_cache unlikely tokens scale={scale}", flush=True)
    spec = SPECS["bf16_ragged"]
    w, g = _make(spec)
    Wg = (g["W"].float() * scale).to(torch.bfloat16)
    # behaviour weights: drifted by ~10 nats per logit in the first case, the current ones in the second
    Wold = (g["W_old"].float() * scale).to(torch.bfloat16) if scale < 100 else Wg
    gen = torch.Generator().manual_seed(5)
    tokens = torch.randint(0, spec.V, tuple(g["tokens"].shape), generator=gen, dtype=torch.int32).cuda()
    N = tokens.shape[0]
    coef = np.random.default_rng(6).normal(size=N).astype(np.float32)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], Wold, tokens, g["mask"])
    H, _, _, mask = _oracle_inputs(w)
    ref = orc.iw_pg_loss_fwd_bwd(H, _np(Wg), tokens.cpu().numpy(), mask, _np(logp_b), _np(w["rewards"]),
                                 _np(w["group_ids"]), w["K"], coef_override=coef)
    spread = -ref["logp_cur"][mask != 0]
    assert (spread.max() < 70) if scale < 100 else (np.median(spread) > 100)
    logp_ok = lambda out: np.all(np.abs(_np(out.logp_cur) - ref["logp_cur"]) <= 2e-5 + 2e-6 * np.abs(ref["logp_cur"]))
    for cache in (True, False):
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], Wg, tokens, g["mask"], logp_b, g["rewards"], g["group_ids"],
                                          w["K"], logits_cache=cache, coef_override=torch.from_numpy(coef).cuda())
        torch.cuda.synchronize()
        assert logp_ok(out) and abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
        assert out.dev_status.item() == 0
        _dh_ok(out.dhidden, ref["dH"])
        _dw_ok(out.dW, ref["dW"])
    # no behaviour log-probs: the reference is the sampled token's own logit
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], Wg, tokens, g["mask"], None, g["rewards"], g["group_ids"],
                                      w["K"], logits_cache=True, coef_override=torch.from_numpy(coef).cuda())
    torch.cuda.synchronize()
    assert logp_ok(out)
    if scale < 100:
        assert out.dev_status.item() == 0
        _dh_ok(out.dhidden, ref["dH"])
        _dw_ok(out.dW, ref["dW"])
    else:
        assert out.dev_status.item() == rb.STATUS_LOGIT_RANGE
        assert np.isfinite(_np(out.dhidden)).all() and np.isfinite(_np(out.dW)).all()


def test_logits_cache_sized_for_a_token_bound(rb):
    """opts.max_tokens: a cache of the promised number of tokens (instead of N*T rows) holds the whole
    batch; with the exact count the results are the bits of the unbounded one-chunk cache.  The same
    workspace with a larger promise cannot hold the batch at once any more and the call works through it
    in chunks (same results up to rounding); a broken promise is reported on the device, nothing else."""
    spec = wl.small_spec("bound", "bf16", d=128, V=1000, prompts=6, G=4, len_lo=30, len_hi=200)
    w, g = _make(spec)
    N, T, d = g["hidden"].shape
    M = int(g["mask"].sum().item())
    assert M + 512 < N * T
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    args = (g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], w["K"])
    full_buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=True, max_tokens=N * T)
    full = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=full_buf, logits_cache=True)
    small_buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=True, max_tokens=M)
    assert small_buf.workspace.numel() < full.workspace.numel()
    out = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=small_buf, logits_cache=True, max_tokens=M)
    torch.cuda.synchronize()
    assert out.dev_status.item() == 0
    for k in ("loss", "dW", "logp_cur", "seq_logratio", "adv"):
        assert torch.equal(getattr(out, k), getattr(full, k)), k
    # dHidden cuts a partly filled last round of tiles along the vocabulary, and where it cuts depends on the
    # number of workgroups of the launch, which follows the rows the cache was sized for: another order of summation
    assert _rel(_np(out.dhidden), _np(full.dhidden)) <= 2e-3
    ref_dW, ref_dH = full.dW.clone(), full.dhidden.clone()
    out = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=small_buf, logits_cache=True, max_tokens=M + 600)   # in chunks now
    torch.cuda.synchronize()
    assert out.dev_status.item() == 0 and torch.equal(out.logp_cur, full.logp_cur) and torch.equal(out.loss, full.loss)
    # dW, and dHidden where a launch cut its last round of tiles, are summed in another order
    assert _rel(_np(out.dW), _np(ref_dW)) <= 1e-5
    assert _rel(_np(out.dhidden), _np(ref_dH)) <= 2e-3
    tiny = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=True, max_tokens=M - 300)
    bad = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=tiny, logits_cache=True, max_tokens=M - 300)
    torch.cuda.synchronize()
    assert bad.dev_status.item() & rb.STATUS_TOKEN_BOUND
    assert bad.read_diag()["n_tokens"] == (M - 300 + 255) // 256 * 256        # the rows the cache was sized for


def test_logits_cache_workspace_and_errors(rb):
    spec = SPECS["bf16_small"]
    w, g = _make(spec)
    N, T, d = g["hidden"].shape
    V = g["W"].shape[1]
    need = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, w["K"], rb.DTYPE_BF16)
    least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, w["K"], rb.DTYPE_BF16, minimum=True)
    whole = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, w["K"], rb.DTYPE_BF16, max_tokens=N * T)
    assert least < need == whole                           # the recommended cache holds this small batch at once
    assert rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, w["K"], rb.DTYPE_F32) == 0
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    small = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], workspace_bytes=least - 4096)
    with pytest.raises(rb.RapidError) as e:
        rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"],
                                    g["group_ids"], w["K"], buffers=small, logits_cache=True)
    assert e.value.code == -4


CHUNKY = wl.small_spec("chunky", "bf16", d=136, V=1100, prompts=7, G=3, len_lo=5, len_hi=60, sigma=0.02, reward="uniform")


@pytest.mark.parametrize("size", ["minimum", "middle", "nearly_full"])
def test_cached_backward_in_chunks_of_whole_groups(rb, size):
    """logits_cache = 1 with a workspace whose cache cannot hold the batch: chunks of whole groups, each
    forward-with-store, estimator, dHidden, dW.  With the smallest workspace (a cache of 256 rows: one
    or two groups of three generations per chunk), one in the middle and one a few bytes short of
    the one-chunk size; every output against the oracle, for the default options, normalised gradients
    (the running rescaling of dW and dHidden), the token-level weight, a bf16 dW, accumulation into
    the caller's dW, and the final norm."""
    spec = CHUNKY
    w, g = _make(spec, seed=4)
    N, T, d = g["hidden"].shape
    V, K = spec.V, w["K"]
    least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, minimum=True)
    whole = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, max_tokens=N * T)
    nbytes = {"minimum": least, "middle": (least + whole) // 2, "nearly_full": whole - 256}[size]
    H, W, tok, mask = _oracle_inputs(w)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    args = (g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], K)
    for kw in (dict(), dict(normalized_grads=True), dict(ratio_level=1, coef_mode=1, eta=1.05, normalized_grads=True),
               dict(baseline_mode=2, temperature=0.8)):
        print(f"chunked cache {size}: {kw}", flush=True)
        lb = logp_b if "temperature" not in kw else rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"],
                                                                          temperature=kw["temperature"])[0]
        buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lb, g["rewards"], g["group_ids"], K,
                                          buffers=buf, logits_cache=True, **kw)
        torch.cuda.synchronize()
        ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(lb), _np(w["rewards"]), _np(w["group_ids"]), K, **kw)
        _check_pair(rb, spec, out, ref)
        if kw.get("normalized_grads"):
            assert abs(out.read_diag()["grad_log_scale"] - ref["grad_log_scale"]) <= 1e-3
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), K, normalized_grads=True)
    # bf16 dW, and accumulation into what the caller holds (with normalised gradients: through the staging buffer)
    buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes, dw_dtype=torch.bfloat16)
    out = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=buf, logits_cache=True, normalized_grads=True)
    torch.cuda.synchronize()
    _dw_ok(out.dW, ref["dW"], rel=2.0 ** -6)
    buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
    for norm in (True, False):
        buf.dW.fill_(0.25)
        out = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=buf, logits_cache=True, normalized_grads=norm, accumulate_dw=True)
        torch.cuda.synchronize()
        want = ref["dW"] if norm else ref["dW"] * math.exp(ref["grad_log_scale"])
        err = np.abs(_np(out.dW) - 0.25 - want)
        assert np.all(err <= 3 * 2.0 ** -8 * np.abs(want).max(axis=0, keepdims=True) + 6e-8), norm
    # the final norm on the way in and out
    rng = np.random.default_rng(32)
    x = (g["hidden"].float() * torch.from_numpy(rng.uniform(0.3, 3.0, size=(N, T, 1))).float().cuda()).to(torch.bfloat16)
    wgt = torch.from_numpy(1.0 + 0.2 * rng.normal(size=d)).float().cuda().to(torch.bfloat16)
    eps = float(np.float32(1e-5))
    lb, _ = rb.rapid_logprob_fwd(x, g["W_old"], g["tokens"], g["mask"], rms_weight=wgt, rms_eps=eps)
    buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
    out = rb.rapid_iw_pg_loss_fwd_bwd(x, g["W"], g["tokens"], g["mask"], lb, g["rewards"], g["group_ids"], K, buffers=buf,
                                      logits_cache=True, normalized_grads=True, rms_weight=wgt, rms_eps=eps)
    torch.cuda.synchronize()
    ref = orc.iw_pg_loss_fwd_bwd(_np(x), W, tok, mask, _np(lb), _np(w["rewards"]), _np(w["group_ids"]), K, normalized_grads=True,
                                 rms_weight=_np(wgt), rms_eps=eps, round_normed_hidden=True)
    assert out.dev_status.item() == 0
    assert np.abs(_np(out.logp_cur) - ref["logp_cur"]).max() <= LOGP_ATOL["bf16"]
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dw_ok(out.dW, ref["dW"])
    _dh_ok(out.dhidden, ref["dH"], rel=2.0 ** -5)        # dL/dh stored in bf16, rescaled, then through the norm
    assert _rel(_np(out.drms_weight), ref["d_rms_weight"]) <= GRAD_RTOL["bf16"]


def test_cached_backward_in_chunks_needs_adjacent_groups_that_fit(rb):
    """The two conditions of the chunked cache are checked on the device and reported, nothing else
    happens: members of a group apart in the batch; a group with more tokens than the cache has rows.
    With the one-chunk workspace neither matters."""
    spec = CHUNKY
    w, g = _make(spec, seed=4)
    N, T, d = g["hidden"].shape
    V, K = spec.V, w["K"]
    least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, minimum=True)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    shuffled = g["group_ids"][torch.randperm(N, generator=torch.Generator().manual_seed(0)).cuda()].contiguous()
    one_group = torch.zeros_like(g["group_ids"])
    H, W, tok, mask = _oracle_inputs(w)
    for gid, kk in ((shuffled, K), (one_group, 1)):
        buf = rb.IwPgBuffers(g["hidden"], g["W"], kk, workspace_bytes=least)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], gid, kk,
                                          buffers=buf, logits_cache=True)
        torch.cuda.synchronize()
        assert out.dev_status.item() & rb.STATUS_GROUP_LAYOUT          # the outputs are not usable then; nothing faulted
        whole = rb.IwPgBuffers(g["hidden"], g["W"], kk, logits_cache=True, max_tokens=N * T)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], gid, kk,
                                          buffers=whole, logits_cache=True)
        torch.cuda.synchronize()
        ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(gid), kk)
        _check_pair(rb, spec, out, ref)


@pytest.mark.parametrize("size", ["minimum", "middle", "whole", "recompute"])
def test_generations_without_gradient_are_left_out(rb, size):
    """A group whose rewards are all 0 has A_n = 0 whatever the ratios are (Eq. (5): the weighted baseline of zeros is
    0), so its generations get no gradient; the cached backward puts them last inside their chunk and its two
    gradient contractions stop in front of them.  Every output must be what the oracle, which leaves nothing out,
    gives: zero groups at the start, in the middle (across chunk boundaries) and at the end of the batch, every
    group zero, a coefficient override with zeros, and the baselines' step without a KL term; also against the
    same call with the skipping switched off.  "recompute": the backward that regenerates the logits does the
    same with the batch as its one chunk."""
    spec = CHUNKY
    w, g = _make(spec, seed=9)
    N, T, d = g["hidden"].shape
    V, K = spec.V, w["K"]
    least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, minimum=True)
    whole = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, max_tokens=N * T)
    cache = size != "recompute"
    nbytes = {"minimum": least, "middle": (least + whole) // 2, "whole": whole, "recompute": None}[size]
    H, W, tok, mask = _oracle_inputs(w)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    gid = _np(w["group_ids"]).astype(np.int64)
    R0 = _np(w["rewards"]).astype(np.float32)

    def run(rewards, **kw):
        buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, torch.from_numpy(rewards).cuda(),
                                          g["group_ids"], K, buffers=buf, logits_cache=cache, **kw)
        torch.cuda.synchronize()
        return out

    for zero_groups in ([0], [2, 3], [K - 1], [0, 1, 3, 4, K - 1], list(range(K))):
        print(f"zero-reward groups {zero_groups}, window {size}", flush=True)
        R = R0.copy()
        R[np.isin(gid, zero_groups)] = 0.0
        for kw in (dict(), dict(normalized_grads=True, ratio_level=1)):
            out = run(R, **kw)
            ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), R, _np(w["group_ids"]), K, **kw)
            ref["slack"] = pb.coefficient_slack(ref, R, mask)
            idle_rows = np.isin(gid, zero_groups)
            assert np.all(ref["dH"][idle_rows] == 0.0) and np.all(_np(out.dhidden)[idle_rows] == 0.0)
            if len(zero_groups) == K:              # nothing carries gradient: exact zeros everywhere
                assert out.loss.item() == 0.0 and not _np(out.dW).any() and not _np(out.dhidden).any()
                assert np.abs(_np(out.logp_cur) - ref["logp_cur"]).max() <= LOGP_ATOL["bf16"]
                assert out.read_diag()["n_tokens"] == ref["n_tokens"] and out.dev_status.item() == 0
                continue
            _check_pair(rb, spec, out, ref)
            rb.rapid_set_tuning(19, 0)             # the same call with every generation in the contractions
            try:
                full = run(R, **kw)
            finally:
                rb.rapid_set_tuning(19, 1)
            assert torch.equal(full.logp_cur, out.logp_cur) and full.loss.item() == out.loss.item()
            assert _rel(_np(out.dW), _np(full.dW)) <= 2e-3 and _rel(_np(out.dhidden), _np(full.dhidden)) <= 2e-3
    # a coefficient override with zeros decides by itself (here: two generations of different groups, rewards untouched)
    coef = np.linspace(-1.0, 1.0, N).astype(np.float32) / N
    coef[[1, 5, N - 1]] = 0.0
    out = run(R0, coef_override=torch.from_numpy(coef).cuda())
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), R0, _np(w["group_ids"]), K, coef_override=coef)
    assert out.dev_status.item() == 0 and abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dh_ok(out.dhidden, ref["dH"])
    _dw_ok(out.dW, ref["dW"])
    assert not _np(out.dhidden)[[1, 5, N - 1]].any()
    # the baselines' step: without a KL term (DAPO) a zero group is idle; with one (GRPO) every token carries gradient
    R = R0.copy()
    R[np.isin(gid, [1, 4])] = 0.0
    ref_w = (g["W"].float() + 0.01 * torch.randn(g["W"].shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))).to(torch.bfloat16)
    logp_ref, _ = rb.rapid_logprob_fwd(g["hidden"], ref_w, g["tokens"], g["mask"])
    for variant in ("dapo", "grpo"):
        buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
        out = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, logp_ref, torch.from_numpy(R).cuda(),
                                            g["group_ids"], K, variant=variant, buffers=buf, logits_cache=cache)
        torch.cuda.synchronize()
        co = rb.clip_pg_default_opts(variant)
        o = orc.clipped_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(logp_ref), R, _np(w["group_ids"]), K,
                                        eps_low=co.eps_low, eps_high=co.eps_high, kl_beta=co.kl_beta, norm_mode=co.norm_mode)
        assert out.dev_status.item() == 0 and abs(out.loss.item() - o["loss"]) <= LOSS_RTOL * abs(o["loss"]), variant
        assert _rel(_np(out.dW), o["dW"]) <= GRAD_RTOL["bf16"] and _rel(_np(out.dhidden), o["dH"]) <= GRAD_RTOL["bf16"], variant
        if variant == "dapo":
            assert not _np(out.dhidden)[np.isin(gid, [1, 4])].any()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_short_generations(rb, dtype):
    """Nine thousand generations in three thousand groups: the prefix sum over the generations takes more than one
    sweep of its block, and the per-group reductions go over each group's run of the batch (groups adjacent) or,
    with the group ids shuffled, over the whole batch; every output against the oracle, in both backward modes."""
    spec = wl.small_spec("many", dtype, d=16, V=40, prompts=3000, G=3, len_lo=1, len_hi=3, sigma=0.05, reward="uniform")
    w, g = _make(spec, seed=2)
    H, W, tok, mask = _oracle_inputs(w)
    K = w["K"]
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    shuffled = g["group_ids"][torch.randperm(len(g["group_ids"]), generator=torch.Generator().manual_seed(1)).cuda()].contiguous()
    for gid in (g["group_ids"], shuffled):
        ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(gid), K)
        ref["slack"] = pb.coefficient_slack(ref, _np(w["rewards"]), mask)
        for cache in ((False, True) if dtype == "bf16" else (False,)):
            print(f"many generations {dtype}, cache {cache}, shuffled {gid is shuffled}", flush=True)
            out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], gid, K,
                                              logits_cache=cache)
            torch.cuda.synchronize()
            _check_pair(rb, spec, out, ref)


def _random_specs(count, seed):
    """Seeded shapes off every tile boundary: d a multiple of 8 (bf16) or anything (f32), V from a handful to a few
    tiles, group counts and lengths from one token up."""
    rng = np.random.default_rng(seed)
    specs = []
    for i in range(count):
        dtype = "bf16" if i % 3 else "f32"
        d = int(rng.integers(1, 41)) * 8 if dtype == "bf16" else int(rng.integers(1, 90))
        V = int(rng.choice([rng.integers(2, 40), rng.integers(40, 600), rng.integers(600, 1400)]))
        prompts, G = int(rng.integers(1, 7)), int(rng.integers(1, 6))
        lo = int(rng.integers(1, 30))
        hi = lo + int(rng.integers(0, 90))
        specs.append(wl.small_spec(f"random{i}", dtype, d=d, V=V, prompts=prompts, G=G, len_lo=lo, len_hi=hi,
                                   sigma=float(rng.choice([0.0, 0.01, 0.05])), reward=str(rng.choice(["bernoulli", "uniform"]))))
    return specs


@pytest.mark.parametrize("spec", _random_specs(18, seed=2024), ids=lambda s: f"{s.name}-{s.dtype}-d{s.d}-V{s.V}-{s.prompts}x{s.G}-L{s.len_lo}-{s.len_hi}")
def test_random_shapes(rb, spec):
    """A seeded sweep of small shapes that sit on no tile boundary: every output of the fused call against the
    oracle, with the regenerating backward and (bf16) with the cache at its smallest window and at its default size,
    options drawn per shape."""
    rng = np.random.default_rng(spec.d * 1000 + spec.V)
    kw = dict(baseline_mode=int(rng.integers(0, 3)), coef_mode=int(rng.integers(0, 2)), eta=float(rng.choice([1.2, 2.0, math.inf])),
              normalized_grads=bool(rng.integers(0, 2)))
    if spec.dtype == "bf16" and rng.integers(0, 3) == 0:
        kw["ratio_level"] = 1
    print(f"random shape {spec} {kw}", flush=True)
    for cache in ((False, True) if spec.dtype == "bf16" else (False,)):
        w, out, ref = _run_pair(rb, spec, seed=7, logits_cache=cache, **kw)
        _check_pair(rb, spec, out, ref)
        if kw["normalized_grads"]:
            assert abs(out.read_diag()["grad_log_scale"] - ref["grad_log_scale"]) <= 1e-3
    if spec.dtype == "bf16":       # smallest window: chunks of whole groups (a group of more than 256 tokens cannot go through it)
        w, g = _make(spec, seed=7)
        lengths = _np(w["mask"]).sum(1).reshape(spec.prompts, spec.G).sum(1)
        if lengths.max() <= 256:
            N, T, d = g["hidden"].shape
            least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, w["K"], rb.DTYPE_BF16, minimum=True)
            logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
            buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], workspace_bytes=least)
            out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"],
                                              w["K"], buffers=buf, logits_cache=True, **kw)
            torch.cuda.synchronize()
            _check_pair(rb, spec, out, ref)


def test_inner_loop_on_synthetic_bandit(rb):
    """Alg. 1's inner loop, H mini-batches of one inference batch: the first step is exactly on-policy,
    staleness grows with the step index, the estimated reward of the policy improves, and a call at
    the weights the loop arrived at still matches the oracle."""
    from paper_2510_03515_amd import iw_grpg as loop
    spec = wl.small_spec("bandit", "bf16", d=128, V=1000, prompts=24, G=4, len_lo=4, len_hi=24, sigma=0.0,
                         tokens_from="cur")
    w, g = _make(spec, seed=1)
    log, summary, W_end = loop.iw_grpg(g, inner_steps=6, lr=0.05)
    log_c, _, W_end_c = loop.iw_grpg(g, inner_steps=6, lr=0.05, logits_cache=True)    # same run on the cached ratios
    assert [r["loss"] for r in log_c][:1] == [r["loss"] for r in log][:1]
    assert max(abs(a["staleness"] - b["staleness"]) for a, b in zip(log, log_c)) < 0.02
    assert _rel(_np(W_end_c), _np(W_end)) < 1e-2
    assert log[0]["staleness"] == 0.0 and log[0]["clip_fraction"] == 0.0 and log[0]["max_abs_s"] == 0.0
    assert abs(log[0]["loss"]) <= 1e-6                 # complete groups, all weights 1: the advantages cancel
    st = [r["staleness"] for r in log]
    assert st[1] > 0 and st[-1] > st[1] and sum(st[3:]) > sum(st[:3])   # grows with the number of inner steps
    assert summary["reward_final_is_estimate"] > summary["reward_behaviour"]
    # one more evaluation at the final weights against the oracle
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], W_end, g["tokens"], g["mask"], logp_b, g["rewards"],
                                      g["group_ids"], w["K"], coef_mode=1)
    torch.cuda.synchronize()
    H, _, tok, mask = _oracle_inputs(w)
    ref = orc.iw_pg_loss_fwd_bwd(H, _np(W_end).astype(np.float64), tok, mask, _np(logp_b), _np(w["rewards"]),
                                 _np(w["group_ids"]), w["K"], coef_mode=1)
    assert np.abs(_np(out.seq_logratio) - ref["seq_logratio"]).max() <= S_ATOL
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dw_ok(out.dW, ref["dW"])
    # the same loop with AdamW as the update: first step on-policy as well, staleness grows, the estimate improves
    log_a, summary_a, _ = loop.iw_grpg(g, inner_steps=6, lr=2e-3, optimizer="adamw")
    assert log_a[0]["staleness"] == 0.0 and log_a[-1]["staleness"] > log_a[1]["staleness"] > 0
    assert summary_a["reward_final_is_estimate"] > summary_a["reward_behaviour"]
    # the update itself: fp32 master, bf16 copy
    m = torch.randn(1000, device="cuda"); gr = torch.randn(1000, device="cuda"); wo = torch.empty(1000, dtype=torch.bfloat16, device="cuda")
    m0 = m.clone()
    rb.rapid_sgd_step(m, gr, 0.5, w_out=wo)
    assert torch.equal(m, m0 - 0.5 * gr) and torch.equal(wo, m.to(torch.bfloat16))


@pytest.mark.parametrize("waves", [4, 8, 16])
def test_other_workgroup_geometries(rb, waves):
    """Every contraction kernel in the 4-, 8- and 16-wave geometry (rapid_set_tuning key 2; by default
    dHidden runs with 4 waves and the others with 8): the same tiles in a different split, same
    tolerances against the oracle."""
    print(f"geometry {waves} waves", flush=True)
    try:
        rb.rapid_set_tuning(2, waves)
        for name in ("bf16_small", "bf16_ragged"):
            w, out, ref = _run_pair(rb, SPECS[name])
            _check_pair(rb, SPECS[name], out, ref)
        w, out, ref = _run_pair(rb, SPECS["bf16_ragged"], layout="vd", logits_cache=True)
        _check_pair(rb, SPECS["bf16_ragged"], out, ref, "vd")
    finally:
        rb.rapid_set_tuning(2, 0)


@pytest.mark.parametrize("variant", [1, 2, 3])
def test_forward_with_k_steps_of_32(rb, variant):
    """Tuning key 21: the logits kernel with K steps of 32 and W from its K-blocked copy, as two 4-wave workgroups
    per CU on 256 x 128 tiles through three LDS stages (1), or as one 8-wave workgroup on 256 x 256 tiles through
    four stages, requests three steps ahead (2), or that with 4 waves of 128 x 128 (3).  Same tolerances against the oracle: the behaviour pass, the fused
    call in both backward modes and layouts, the chunked cache; and the same log-probs, bit for bit, as the
    default kernel (the same products summed in the same order per accumulator)."""
    try:
        base = {}
        for name in ("bf16_small", "bf16_ragged"):
            w, g = _make(SPECS[name])
            base[name] = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])[0].clone()
        rb.rapid_set_tuning(21, variant)
        for name in ("bf16_small", "bf16_ragged"):
            print(f"K steps of 32, variant {variant}: {name}", flush=True)
            w, g = _make(SPECS[name])
            lp, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
            torch.cuda.synchronize()
            assert torch.equal(lp, base[name])
            for cache in (False, True):
                w, out, ref = _run_pair(rb, SPECS[name], logits_cache=cache)
                _check_pair(rb, SPECS[name], out, ref)
        w, out, ref = _run_pair(rb, SPECS["bf16_ragged"], layout="vd", logits_cache=True)
        _check_pair(rb, SPECS["bf16_ragged"], out, ref, "vd")
        # chunks of whole groups at the smallest window
        spec = CHUNKY
        w, g = _make(spec, seed=4)
        N, T, d = g["hidden"].shape
        least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, w["K"], rb.DTYPE_BF16, minimum=True)
        logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
        buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], workspace_bytes=least)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], w["K"],
                                          buffers=buf, logits_cache=True)
        torch.cuda.synchronize()
        H, W, tok, mask = _oracle_inputs(w)
        ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"])
        _check_pair(rb, spec, out, ref)
    finally:
        rb.rapid_set_tuning(21, 0)


@pytest.mark.parametrize("V", [520, 200])
def test_dhidden_cut_last_round(rb, V):
    """dHidden with more tiles than workgroups and a last round that fills a fraction of them: 140 row tiles x 2
    column tiles = 280 tiles on 256 workgroups, 35 per XCD, so each XCD's last round holds 3 tiles, whose contraction
    is cut into segments, written as partial tiles and summed by the reduce pass.  V = 520 is 12 K steps per tile
    (8 segments of one or two steps); V = 200 is 4 (4 segments of one step).  Against
    the oracle in both backward modes, and against the same call with the cut switched off (tuning key 17)."""
    spec = wl.small_spec("dh_cut", "bf16", d=512, V=V, prompts=35, G=4, len_lo=256, len_hi=256, sigma=0.02, reward="uniform")
    w, g = _make(spec, seed=3)
    H, W, tok, mask = _oracle_inputs(w)
    K = w["K"]
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), K)
    ref["slack"] = pb.coefficient_slack(ref, _np(w["rewards"]), mask)
    for cache in (False, True):
        print(f"dHidden cut, V={V}, cache {cache}", flush=True)
        out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], K,
                                          logits_cache=cache, max_tokens=int(mask.sum()))
        torch.cuda.synchronize()
        _check_pair(rb, spec, out, ref)
        dh_cut = out.dhidden.clone()
        try:
            rb.rapid_set_tuning(17, 0)
            out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], K,
                                              logits_cache=cache, max_tokens=int(mask.sum()))
            torch.cuda.synchronize()
        finally:
            rb.rapid_set_tuning(17, 1)
        _check_pair(rb, spec, out, ref)
        # the same products in another order of summation: equal up to the fp32 rounding of the accumulators
        assert _rel(_np(dh_cut), _np(out.dhidden)) <= 2e-3
        assert not torch.equal(dh_cut, out.dhidden) or V == 200


@pytest.mark.parametrize("key,value,default", [(2, 8, 0), (17, 0, 1)])
def test_dw_with_k_steps_of_32(rb, key, value, default):
    """Tuning key 22: the dW kernel with K steps of 32 rows through four LDS stages, requests three steps ahead.  The
    same products are added in the same order per accumulator, so dW must come out bit for bit as from the default
    loop; shapes with one row tile, several, a d padded to 128-wide tiles, and the 35840-row batch of the cut test.  Key 2 = 8
    (with tiles that are cut) or key 17 = 0 (without) keep short contractions from tiles of 128 x 128, which have no such loop."""
    cases = [("bf16_small", SPECS["bf16_small"], 0), ("bf16_ragged", SPECS["bf16_ragged"], 0), ("chunky", CHUNKY, 4),
             ("long", wl.small_spec("dh_cut", "bf16", d=512, V=520, prompts=35, G=4, len_lo=256, len_hi=256, sigma=0.02,
                                    reward="uniform"), 3)]
    for name, spec, seed in cases:
        for cache in (False, True):
            print(f"dW K steps of 32: {name}, cache {cache}, key {key}", flush=True)
            try:
                rb.rapid_set_tuning(key, value)
                w, out, ref = _run_pair(rb, spec, seed=seed, logits_cache=cache)
                base = out.dW.clone()
                rb.rapid_set_tuning(22, 1)
                w, out, ref = _run_pair(rb, spec, seed=seed, logits_cache=cache)
            finally:
                rb.rapid_set_tuning(22, 0)
                rb.rapid_set_tuning(key, default)
            assert torch.equal(out.dW, base)
            _check_pair(rb, spec, out, ref)


def test_dhidden_pacing_is_timing_only(rb):
    """Tuning key 16: the dHidden workgroups meet every so many K steps (a vocabulary of 20 000 makes
    313 steps, so meetings every 64 steps do happen here, with fewer workgroups than CUs; key 17 = 0, because the
    workgroups of cut tiles do not meet): same bits as unpaced, and the result matches the oracle."""
    spec = wl.small_spec("pace", "bf16", d=64, V=20000, prompts=3, G=4, len_lo=20, len_hi=70)
    try:
        rb.rapid_set_tuning(17, 0)
        rb.rapid_set_tuning(16, 64)
        w, out, ref = _run_pair(rb, spec)
        _check_pair(rb, spec, out, ref)
        w, outc, _ = _run_pair(rb, spec, logits_cache=True)
        rb.rapid_set_tuning(16, 0)
        w, out0, _ = _run_pair(rb, spec)
        w, outc0, _ = _run_pair(rb, spec, logits_cache=True)
    finally:
        rb.rapid_set_tuning(16, 0)
        rb.rapid_set_tuning(17, 1)
    assert torch.equal(out.dhidden, out0.dhidden) and torch.equal(out.dW, out0.dW)
    assert torch.equal(outc.dhidden, outc0.dhidden) and torch.equal(outc.dW, outc0.dW)


def test_row_major_w_for_dhidden(rb):
    """Tuning key 14 = 0: dHidden from the row-major copy of W instead of the tile-blocked one: same bits."""
    spec = SPECS["bf16_ragged"]
    w, out, ref = _run_pair(rb, spec)
    try:
        rb.rapid_set_tuning(14, 0)
        w2, out2, _ = _run_pair(rb, spec)
    finally:
        rb.rapid_set_tuning(14, 1)
    assert torch.equal(out.dhidden, out2.dhidden) and torch.equal(out.dW, out2.dW)


@pytest.mark.parametrize("mode", [dict(), dict(logits_cache=True, ratio_level=1, coef_mode=1),
                                  dict(logits_cache=True, normalized_grads=True, chunks=True)])
def test_hip_graph_replay_matches_eager(rb, mode):
    """The fused call only enqueues kernels on the caller's stream (no allocation, no host read of
    device data, no memset nodes), so it can be captured into a HIP graph; every replay, with eager
    work in between, gives the bits of the eager call (default options; the cache with the
    token-level weight; the cache at its smallest window, i.e. several chunks of whole groups whose
    sizes only the device knows, with the running rescale of normalised gradients)."""
    mode = dict(mode)
    chunks = mode.pop("chunks", False)
    spec = CHUNKY if chunks else SPECS["bf16_ragged"]
    w, g = _make(spec)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    if chunks:
        N, T, d = g["hidden"].shape
        least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, w["K"], rb.DTYPE_BF16, minimum=True)
        buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], workspace_bytes=least)
    else:
        buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=mode.get("logits_cache", False))
    call = lambda: rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"],
                                               g["group_ids"], w["K"], buffers=buf, **mode)
    call()
    torch.cuda.synchronize()
    ref = {k: getattr(buf, k).clone() for k in ("loss", "dhidden", "dW", "logp_cur", "seq_logratio", "adv")}
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()                                   # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call()
    torch.cuda.synchronize()
    for rep in range(3):
        for k in ref:                            # eager work between replays: wipe the outputs
            getattr(buf, k).fill_(float("nan") if getattr(buf, k).is_floating_point() else 0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k, v in ref.items():
            assert torch.equal(getattr(buf, k), v), (rep, k)


def test_fused_shuffled_groups_mask_holes_and_bad_values(rb):
    """Groups in arbitrary order with unequal sizes and an empty group, a mask with holes (not just
    right padding), and non-finite rewards / behaviour log-probs (flagged in dev_status and counted
    as 0): the fused call against the oracle on the same inputs with the bad values zeroed."""
    spec = SPECS["bf16_ragged"]
    w, g = _make(spec, seed=5)
    rng = np.random.default_rng(11)
    N, T = w["mask"].shape
    K = w["K"] + 1                                            # group K-1 stays empty
    gid = rng.integers(0, K - 1, size=N).astype(np.int32)
    mask = (w["mask"].numpy() & (rng.random((N, T)) < 0.8)).astype(np.uint8)
    mask[0, :] = 0
    mask[0, 5] = 1                                            # a generation with a single, isolated token
    mask_g = torch.from_numpy(mask).cuda()
    gid_g = torch.from_numpy(gid).cuda()
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], mask_g)
    H, W, tok, _ = _oracle_inputs(w)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], mask_g, logp_b, g["rewards"], gid_g, K)
    torch.cuda.synchronize()
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), gid, K)
    assert out.dev_status.item() == 0
    assert np.abs(_np(out.seq_logratio) - ref["seq_logratio"]).max() <= S_ATOL
    assert np.allclose(_np(out.adv), ref["adv"], atol=1e-3)
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dh_ok(out.dhidden, ref["dH"])
    _dw_ok(out.dW, ref["dW"])
    assert torch.all(out.dhidden[mask_g == 0] == 0)
    assert out.read_diag()["n_tokens"] == int(mask.sum())
    # non-finite reward and behaviour log-prob: flagged, treated as 0
    rewards = g["rewards"].clone()
    rewards[3] = float("nan")
    lb = logp_b.clone()
    n_bad, t_bad = np.argwhere(mask == 1)[7]
    lb[n_bad, t_bad] = float("inf")
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], mask_g, lb, rewards, gid_g, K)
    torch.cuda.synchronize()
    st = out.dev_status.item()
    assert st & rb.STATUS_NONFINITE_REWARD and st & rb.STATUS_NONFINITE_LOGP
    r0 = _np(w["rewards"]).copy(); r0[3] = 0.0
    assert torch.isfinite(out.dW).all() and torch.isfinite(out.loss).all()
    # the bad log-prob's token contributes a log ratio of 0: same as a behaviour log-prob equal to the current one
    lb0 = _np(logp_b).copy(); lb0[n_bad, t_bad] = _np(out.logp_cur)[n_bad, t_bad]
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, lb0, r0, gid, K)
    assert np.abs(_np(out.seq_logratio) - ref["seq_logratio"]).max() <= S_ATOL
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])
    _dw_ok(out.dW, ref["dW"])


# ----------------------------------------------------------------------------- baselines' loss steps
def _clip_inputs(rb, spec, seed, ref_shift=0.02, temperature=1.0):
    """Old-policy log-probs from the workload's W_old; reference log-probs from a third set of weights
    (the policy before the first update, further away than the old policy)."""
    w, g = _make(spec, seed)
    gen = torch.Generator().manual_seed(100 + seed)
    W_ref = (w["W_old"].float() + ref_shift * torch.randn(w["W"].shape, generator=gen)).to(w["W"].dtype).cuda()
    # the old policy a few updates away, so that token ratios leave the clip range on both sides
    W_old = (w["W_old"].float() + 0.03 * torch.randn(w["W"].shape, generator=gen)).to(w["W"].dtype).cuda()
    lp_old, _ = rb.rapid_logprob_fwd(g["hidden"], W_old, g["tokens"], g["mask"], temperature=temperature)
    lp_ref, _ = rb.rapid_logprob_fwd(g["hidden"], W_ref, g["tokens"], g["mask"], temperature=temperature)
    return w, g, lp_old, lp_ref


def _check_clip(rb, spec, w, out, ref, dtype_tol):
    assert out.dev_status.item() == 0
    assert np.abs(_np(out.logp_cur) - ref["logp_cur"]).max() <= LOGP_ATOL[spec.dtype]
    assert np.allclose(_np(out.adv), ref["adv"], atol=1e-5, rtol=1e-5)
    assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * max(abs(ref["loss"]), 1e-30), (out.loss.item(), ref["loss"])
    # what the float storage of the current log-probs may do to each token's coefficient (parity_bounds.py)
    mask = _np(w["mask"])
    tok_slack, col_slack = pb.token_coefficient_slack(ref["coef_of_logp"], ref["logp_cur"], mask, _np(w["tokens"]), spec.V)
    rel = pb.REL[spec.dtype] if dtype_tol is None else dtype_tol
    got_dh, got_dw = _np(out.dhidden), _np(out.dW)
    assert _rel(got_dh, ref["dH"]) <= GRAD_RTOL[spec.dtype] and _rel(got_dw, ref["dW"]) <= GRAD_RTOL[spec.dtype]
    pb.assert_dhidden_close(got_dh, ref["dH"], spec.dtype, rel + tok_slack[:, :, None])
    pb.assert_dw_close(got_dw, ref["dW"], spec.dtype, rel + col_slack[None, :])
    assert np.all(_np(out.dhidden)[_np(w["mask"]) == 0] == 0.0)
    dg = rb.read_clip_diag(out)
    assert dg["n_tokens"] == ref["n_tokens"] and dg["n_sequences"] == len(ref["adv"])
    # the clip decision is taken from float log-probs on one side and float64 ones on the other: tokens whose
    # ratio is within 1e-5 of a clip boundary may fall either way
    r = np.exp(ref["logp_cur"] - ref["logp_old"])[_np(w["mask"]) != 0]
    near = int(((np.abs(r - (1 - ref["eps"][0])) < 1e-5) | (np.abs(r - (1 + ref["eps"][1])) < 1e-5)).sum())
    assert abs(dg["n_clipped"] - round(ref["clip_fraction"] * ref["n_tokens"])) <= near
    assert abs(dg["mean_kl"] - ref["mean_kl"]) <= 1e-5 + 1e-3 * ref["mean_kl"]


@pytest.mark.parametrize("name", ["f32_cfg0", "f32_ragged", "bf16_small", "bf16_ragged"])
@pytest.mark.parametrize("variant", ["grpo", "dapo"])
def test_clip_pg_loss_step(rb, name, variant):
    """The loss step of the GRPO and DAPO baselines on the same kernels: every output against the
    oracle, with the variants' default options and with others (sample std, no advantage epsilon,
    temperature, loss scale, the other normalisation), in both backward modes and both layouts."""
    spec = SPECS[name]
    print(f"clip pg {variant} {name}", flush=True)
    for kw in (dict(), dict(std_ddof=1, adv_eps=0.0, loss_scale=0.5), dict(norm_mode=1 if variant == "grpo" else 0, eps_high=0.1),
               dict(temperature=0.8)):
        temp = kw.get("temperature", 1.0)
        w, g, lp_old, lp_ref = _clip_inputs(rb, spec, seed=2, temperature=temp)
        H, W, tok, mask = _oracle_inputs(w)
        o = rb.clip_pg_default_opts(variant)
        okw = dict(eps_low=o.eps_low, eps_high=o.eps_high, kl_beta=o.kl_beta, norm_mode=o.norm_mode, adv_eps=o.adv_eps,
                   std_ddof=o.std_ddof)
        okw.update(kw)
        ref = orc.clipped_pg_loss_fwd_bwd(H, W, tok, mask, _np(lp_old), _np(lp_ref), _np(w["rewards"]), _np(w["group_ids"]),
                                          w["K"], **okw)
        ref["logp_old"], ref["eps"] = _np(lp_old), (okw["eps_low"], okw["eps_high"])
        ckw = {k: v for k, v in okw.items() if k in ("eps_low", "eps_high", "kl_beta", "norm_mode", "loss_scale")}
        ref["coef_of_logp"] = lambda lp, ckw=ckw, ref=ref: orc.clipped_token_coefficients(
            lp, _np(lp_old), _np(lp_ref), mask, ref["adv"], **ckw)[0]
        assert 0.0 < ref["clip_fraction"] < 0.9
        for cache in ((False, True) if spec.dtype == "bf16" else (False,)):
            out = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lp_old, lp_ref, g["rewards"],
                                                g["group_ids"], w["K"], variant=variant, logits_cache=cache, **kw)
            torch.cuda.synchronize()
            _check_clip(rb, spec, w, out, ref, None)
    if spec.dtype == "bf16":      # [V, d] weights, bf16 dW, accumulation
        Wt = g["W"].t().contiguous()
        buf = rb.IwPgBuffers(g["hidden"], Wt, w["K"], w_layout=rb.W_VD, dw_dtype=torch.bfloat16)
        out = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], Wt, g["tokens"], g["mask"], lp_old, lp_ref, g["rewards"], g["group_ids"],
                                            w["K"], variant=variant, buffers=buf, w_layout=rb.W_VD, temperature=0.8)
        torch.cuda.synchronize()
        _dw_ok(_np(out.dW).T, ref["dW"], rel=2.0 ** -6)
        assert abs(out.loss.item() - ref["loss"]) <= LOSS_RTOL * abs(ref["loss"])


def test_clip_pg_special_cases_and_chunks(rb):
    """Equal policies: every ratio is exactly 1, nothing clips, the KL term vanishes against itself, and
    the gradients are those of the plain group-relative gradient with normalised advantages (the oracle's
    backward with -omega A_n); logp_old = NULL is the same call.  A non-finite stored log-prob is flagged.
    And the chunked cache: same results from chunks of whole groups."""
    spec = CHUNKY
    w, g = _make(spec, seed=6)
    H, W, tok, mask = _oracle_inputs(w)
    N, T, d = g["hidden"].shape
    K = w["K"]
    cur, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    a = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], cur, cur, g["rewards"], g["group_ids"], K)
    torch.cuda.synchronize()
    dga = rb.read_clip_diag(a)
    assert dga["n_clipped"] == 0 and dga["mean_kl"] == 0.0 and torch.equal(a.logp_cur, cur)
    ga = orc.normalized_group_advantage(_np(w["rewards"]), _np(w["group_ids"]), K)
    L = mask.sum(1)
    coef = -(ga["adv"] / (N * L))[:, None] * (mask != 0)
    dH, dW = orc.backward(H, W, tok, mask, coef)
    _dh_ok(a.dhidden, dH)
    _dw_ok(a.dW, dW)
    assert abs(a.loss.item() - (-(ga["adv"]).mean())) <= 1e-6
    b = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], None, None, g["rewards"], g["group_ids"], K,
                                      variant="dapo", norm_mode=0)
    torch.cuda.synchronize()
    assert torch.equal(a.dW, b.dW) and torch.equal(a.dhidden, b.dhidden) and torch.equal(a.loss, b.loss)
    bad = cur.clone()
    n_bad, t_bad = np.argwhere(mask == 1)[5]
    bad[n_bad, t_bad] = float("nan")
    c = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], bad, cur, g["rewards"], g["group_ids"], K)
    torch.cuda.synchronize()
    assert c.dev_status.item() & rb.STATUS_NONFINITE_LOGP and torch.isfinite(c.dW).all() and torch.isfinite(c.loss).all()
    # chunks of whole groups
    w, g, lp_old, lp_ref = _clip_inputs(rb, spec, seed=6)
    least = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, K, rb.DTYPE_BF16, minimum=True)
    for variant in ("grpo", "dapo"):
        o = rb.clip_pg_default_opts(variant)
        ref = orc.clipped_pg_loss_fwd_bwd(H, W, tok, mask, _np(lp_old), _np(lp_ref), _np(w["rewards"]), _np(w["group_ids"]), K,
                                          eps_low=o.eps_low, eps_high=o.eps_high, kl_beta=o.kl_beta, norm_mode=o.norm_mode)
        ref["logp_old"], ref["eps"] = _np(lp_old), (o.eps_low, o.eps_high)
        ref["coef_of_logp"] = lambda lp, o=o, ref=ref: orc.clipped_token_coefficients(
            lp, _np(lp_old), _np(lp_ref), mask, ref["adv"], o.eps_low, o.eps_high, o.kl_beta, o.norm_mode)[0]
        buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=least)
        out = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lp_old, lp_ref, g["rewards"],
                                            g["group_ids"], K, variant=variant, buffers=buf, logits_cache=True)
        torch.cuda.synchronize()
        _check_clip(rb, spec, w, out, ref, None)


# up to 4096 generations each one works its group out by itself, above a launch does it per group; several waves per generation from
# 512 positions on
@pytest.mark.parametrize("dtype,prompts,G,len_hi", [("f32", 6, 5, 24), ("f32", 4, 3, 600), ("f32", 1024, 4, 2), ("f32", 1366, 3, 2), ("bf16", 12, 4, 24),
                                                    ("bf16", 1366, 3, 2)])
@pytest.mark.parametrize("groups", ["adjacent", "scattered", "one", "faulty"])
def test_clip_pg_groups_anywhere(rb, dtype, prompts, G, len_hi, groups):
    """Groups that are one run of the batch, scattered ones, the whole batch as one group; "faulty": scattered, with group ids out of
    range and rewards that are not finite, which are flagged and count as no group (advantage 0) and as 0.  Every output against
    the oracle, in both backward modes, and adjacent groups through the smallest cache."""
    spec = wl.small_spec("clip_groups", dtype, d=16, V=40, prompts=prompts, G=G, len_lo=max(1, len_hi // 3), len_hi=len_hi, reward="uniform")
    w, g, lp_old, lp_ref = _clip_inputs(rb, spec, seed=5)
    H, W, tok, mask = _oracle_inputs(w)
    N, T, d = g["hidden"].shape
    K = w["K"]
    rng = np.random.default_rng(N)
    gid, R = _np(w["group_ids"]).astype(np.int32), _np(w["rewards"]).astype(np.float32)
    if groups == "one":
        gid, K = np.zeros(N, np.int32), 1
    elif groups != "adjacent":
        gid = rng.permutation(gid)
    ref_gid, ref_R, ref_K, bits = gid.copy(), R.copy(), K, 0
    if groups == "faulty":
        gid, R = gid.copy(), R.copy()
        lost = rng.choice(N, 5, replace=False)                      # each a group of its own for the oracle: advantage 0
        gid[lost] = [-1, K, -7, K + 3, 2 ** 31 - 1]
        ref_gid[lost] = K + np.arange(5)
        ref_K = K + 5
        odd = rng.choice(np.setdiff1d(np.arange(N), lost), 3, replace=False)
        R[odd] = [np.nan, np.inf, -np.inf]
        ref_R[odd] = 0.0
        bits = rb.STATUS_BAD_GROUP | rb.STATUS_NONFINITE_REWARD
    gid_g, R_g = torch.from_numpy(gid).cuda(), torch.from_numpy(R).cuda()
    for variant in ("grpo", "dapo"):
        o = rb.clip_pg_default_opts(variant)
        ref = orc.clipped_pg_loss_fwd_bwd(H, W, tok, mask, _np(lp_old), _np(lp_ref), ref_R, ref_gid, ref_K, eps_low=o.eps_low,
                                          eps_high=o.eps_high, kl_beta=o.kl_beta, norm_mode=o.norm_mode)
        ref["logp_old"], ref["eps"] = _np(lp_old), (o.eps_low, o.eps_high)
        ref["coef_of_logp"] = lambda lp, o=o, ref=ref: orc.clipped_token_coefficients(
            lp, _np(lp_old), _np(lp_ref), mask, ref["adv"], o.eps_low, o.eps_high, o.kl_beta, o.norm_mode)[0]
        modes = [(False, None)]
        if dtype == "bf16":
            modes.append((True, None))
            if groups == "adjacent":
                modes.append((True, rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, K, rb.DTYPE_BF16, minimum=True)))
        for cache, nbytes in modes:
            print(f"clip groups {dtype} {N} x {T} {groups} {variant} cache {cache} workspace {nbytes}", flush=True)
            buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes, logits_cache=cache)
            out = rb.rapid_clip_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], lp_old, lp_ref, R_g, gid_g, K,
                                                variant=variant, buffers=buf, logits_cache=cache)
            torch.cuda.synchronize()
            assert out.dev_status.item() == bits
            out.dev_status.zero_()
            _check_clip(rb, spec, w, out, ref, None)


def test_clip_pg_time_of_one_large_group(rb):
    """Advantages are linear work: 32 768 generations of one token in one group take about as long as in groups of four (3.5 times
    while every generation looked through the whole group)."""
    N = 32768
    gen = torch.Generator(device="cuda").manual_seed(7)
    hidden = torch.randn((N, 1, 16), generator=gen, device="cuda")
    W = torch.randn((16, 40), generator=gen, device="cuda")
    tokens = torch.randint(0, 40, (N, 1), generator=gen, device="cuda", dtype=torch.int32)
    mask = torch.ones((N, 1), dtype=torch.uint8, device="cuda")
    lp, _ = rb.rapid_logprob_fwd(hidden, W, tokens, mask)
    rewards = torch.rand(N, generator=gen, device="cuda")

    def microseconds(K):
        gid = (torch.arange(N, device="cuda") * K // N).to(torch.int32)
        buf = rb.IwPgBuffers(hidden, W, K)
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                rb.rapid_clip_pg_loss_fwd_bwd(hidden, W, tokens, mask, lp, lp, rewards, gid, K, buffers=buf)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 5 * 1e3)
        return min(times)
    fours, one = microseconds(N // 4), microseconds(1)
    print(f"clip step of {N} generations: groups of four {fours:.0f} us, one group {one:.0f} us", flush=True)
    assert one <= 2.0 * fours


def test_seq_logratio_and_adamw_entry_points(rb):
    """The ratio reduction as a call of its own (arbitrary masks, a non-finite stored log-prob), and the
    AdamW update of the inner loop over a few steps, both against the oracle."""
    rng = np.random.default_rng(51)
    N, T = 37, 301
    cur = (-rng.random((N, T)) * 12).astype(np.float32)
    beh = (cur + rng.normal(size=(N, T)).astype(np.float32) * 0.3).astype(np.float32)
    mask = (rng.random((N, T)) < 0.7).astype(np.uint8)
    mask[3] = 0
    s, tok = rb.rapid_seq_logratio(torch.from_numpy(cur).cuda(), torch.from_numpy(beh).cuda(), torch.from_numpy(mask).cuda(),
                                   want_tokens=True)
    torch.cuda.synchronize()
    assert np.abs(_np(s) - orc.seq_logratio(cur, beh, mask)).max() <= 2e-5          # float storage of a sum of ~200 terms
    # the difference of two floats, formed exactly and rounded to float once: the same bits as the oracle's, rounded
    assert np.array_equal(_np(tok), orc.token_logratio(cur, beh, mask).astype(np.float32).astype(np.float64))
    assert s[3].item() == 0.0
    beh_bad = beh.copy()
    n_bad, t_bad = np.argwhere(mask == 1)[11]
    beh_bad[n_bad, t_bad] = np.inf
    status = torch.zeros(1, dtype=torch.int32).cuda()
    s2, _ = rb.rapid_seq_logratio(torch.from_numpy(cur).cuda(), torch.from_numpy(beh_bad).cuda(), torch.from_numpy(mask).cuda(),
                                  dev_status=status)
    torch.cuda.synchronize()
    beh0 = beh.copy(); beh0[n_bad, t_bad] = cur[n_bad, t_bad]
    assert status.item() & rb.STATUS_NONFINITE_LOGP and np.abs(_np(s2) - orc.seq_logratio(cur, beh0, mask)).max() <= 2e-5
    # AdamW
    n = 5000
    w0 = rng.normal(size=n).astype(np.float32)
    master = torch.from_numpy(w0.copy()).cuda()
    m, v = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    wo = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    w_ref, m_ref, v_ref = w0.astype(np.float64), np.zeros(n), np.zeros(n)
    lr, b1, b2, eps, wd = (float(np.float32(x)) for x in (1e-2, 0.9, 0.999, 1e-8, 0.05))    # the ABI takes floats
    for step in range(1, 5):
        g = (rng.normal(size=n) * 10.0 ** rng.integers(-4, 1)).astype(np.float32)
        rb.rapid_adamw_step(master, torch.from_numpy(g).cuda(), m, v, step, lr, b1, b2, eps, wd, w_out=wo)
        w_ref, m_ref, v_ref = orc.adamw_step(w_ref, g, m_ref, v_ref, step, lr, b1, b2, eps, wd)
        torch.cuda.synchronize()
        assert np.abs(_np(master) - w_ref).max() <= 1e-5 and np.allclose(_np(m), m_ref, rtol=1e-5, atol=1e-9)
        assert np.allclose(_np(v), v_ref, rtol=1e-5, atol=1e-12) and torch.equal(wo, master.to(torch.bfloat16))
