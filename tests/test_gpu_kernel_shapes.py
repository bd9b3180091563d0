"""GPU parity at the sizes where the kernels' tiles, cuts and dispatch rules change over, against the float64 oracle with
the bounds of test_gpu_parity."""
import numpy as np
import pytest
import torch

from paper_2510_03515_amd import workloads as wl
from oracle import rapid_oracle as orc
import parity_bounds as pb
from test_gpu_parity import _check_pair, _dh_ok, _dw_ok, _make, _np, _oracle_inputs, _rel, _run_pair, rb  # noqa: F401  (rb is the library fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,V,prompts,length", [
    (50, 1000, 11, 65),     # logits in 64 x 64 tiles with remainders, dHidden and dW in 16 x 16 tiles, contraction shared out
    (260, 1100, 11, 65),    # dHidden and dW in 32 x 32 tiles
    (520, 3700, 2, 10),     # dW in 64 x 64 tiles, logits in 32 x 32 tiles, fewer rows than a step of the contraction
    (3, 17, 1, 2),          # everything smaller than one tile and one step
])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("min_ws", [False, True])
def test_fp64_matrix_tiles(rb, d, V, prompts, length, layout, min_ws):
    print(f"fp64 tiles d {d} V {V} rows {prompts * 3 * length} {layout} min_ws {min_ws}", flush=True)
    spec = wl.small_spec("f64_tiles", "f32", d=d, V=V, prompts=prompts, G=3, len_lo=max(1, length - 3), len_hi=length, reward="uniform")
    w, out, ref = _run_pair(rb, spec, layout=layout, min_ws=min_ws)
    _check_pair(rb, spec, out, ref, layout)


@pytest.mark.parametrize("d,V,prompts,length", [
    (64, 2100, 1, 40),       # one tile of dHidden, its contraction cut into many segments
    (640, 1300, 5, 60),      # a few tiles, fewer than workgroups, none of them ragged in d
    (384, 3000, 2, 30),      # more tiles along d than rows
    (136, 70, 2, 30),        # a contraction of two steps: nothing to cut
])
@pytest.mark.parametrize("cache", [False, True])
def test_dhidden_of_few_tiles(rb, d, V, prompts, length, cache):
    print(f"dHidden of few tiles d {d} V {V} rows {prompts * 3 * length} cache {cache}", flush=True)
    spec = wl.small_spec("few_tiles", "bf16", d=d, V=V, prompts=prompts, G=3, len_lo=length - 3, len_hi=length, reward="uniform")
    w, out, ref = _run_pair(rb, spec, logits_cache=cache)
    _check_pair(rb, spec, out, ref)


def test_dhidden_pacing_over_whole_rounds(rb):
    """280 tiles on 256 workgroups: the whole round meets every 4 of its 9 K steps (tuning key 16), the cut last round
    does not; same bits as unpaced."""
    spec = wl.small_spec("pace_whole", "bf16", d=512, V=520, prompts=35, G=4, len_lo=256, len_hi=256, sigma=0.02, reward="uniform")
    got = []
    try:
        for every in (4, 0):
            rb.rapid_set_tuning(16, every)
            w, out, ref = _run_pair(rb, spec)
            _check_pair(rb, spec, out, ref)
            got.append(out.dhidden.clone())
    finally:
        rb.rapid_set_tuning(16, 0)
    assert torch.equal(got[0], got[1])


def _dw_in_every_form(rb, w, layout, cache):
    """dW rounded to bf16 and added to what is there, against plain fp32 dW of the same call."""
    g = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in w.items()}
    lay = rb.W_DV if layout == "dv" else rb.W_VD
    W = g["W"] if layout == "dv" else g["W"].t().contiguous()
    args = (g["hidden"], W, g["tokens"], g["mask"], None, g["rewards"], g["group_ids"], w["K"])
    base = rb.rapid_iw_pg_loss_fwd_bwd(*args, w_layout=lay, logits_cache=cache).dW
    buf = rb.IwPgBuffers(g["hidden"], W, w["K"], lay, dw_dtype=torch.bfloat16, logits_cache=cache)
    half = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=buf, w_layout=lay, logits_cache=cache).dW
    assert torch.equal(half, base.to(torch.bfloat16))                       # one rounding of the same sum
    buf = rb.IwPgBuffers(g["hidden"], W, w["K"], lay, logits_cache=cache)
    old = torch.randn_like(buf.dW)
    buf.dW.copy_(old)
    added = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=buf, w_layout=lay, logits_cache=cache, accumulate_dw=True).dW
    assert torch.equal(added, old + base)


@pytest.mark.parametrize("d,V", [(256, 1024), (264, 1027), (72, 259)])     # whole tiles; rows off 16 bytes and ragged tiles
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("cache", [False, True])
def test_dw_leaves_in_every_form(rb, d, V, layout, cache):
    """dW as fp32, rounded to bf16, and added to what is there, from one launch and (smallest workspace) from several."""
    spec = wl.small_spec("dw_store", "bf16", d=d, V=V, prompts=6, G=3, len_lo=20, len_hi=60, reward="uniform")
    for min_ws in (False, True):
        print(f"dW forms d {d} V {V} {layout} cache {cache} min_ws {min_ws}", flush=True)
        w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache, min_ws=min_ws)
        _check_pair(rb, spec, out, ref, layout)
        w, half, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache, min_ws=min_ws, dw_dtype=torch.bfloat16)
        assert torch.equal(half.dW, out.dW.to(torch.bfloat16))              # one rounding of the same sum
    _dw_in_every_form(rb, w, layout, cache)


@pytest.mark.parametrize("d,V", [(64, 512), (72, 264), (200, 1000), (328, 776), (8, 8), (136, 1003)])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("cache", [False, True])
def test_w_read_in_place(rb, d, V, layout, cache):
    """The head read in place, as small batches do, at whole tiles and steps and past their ends: log-probs bit for bit those
    from the packed copies (tuning key 2 = 8: the same geometry for the logits), gradients within the oracle's bounds
    ([d, V] with V = 1003 is never read in place)."""
    print(f"W in place d {d} V {V} {layout} cache {cache}", flush=True)
    spec = wl.small_spec("in_place", "bf16", d=d, V=V, prompts=5, G=3, len_lo=5, len_hi=70, reward="uniform")
    got = []
    try:
        for waves in (0, 8):
            rb.rapid_set_tuning(2, waves)
            w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache)
            _check_pair(rb, spec, out, ref, layout)
            got.append(out.logp_cur.clone())
    finally:
        rb.rapid_set_tuning(2, 0)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("d,V,prompts,length", [
    (448, 1321, 5, 70),      # ragged vocabulary; more rows than one chunk of the smallest workspace
    (456, 512, 1, 40),       # whole workgroups of columns, few rows
    (512, 130, 6, 64),       # less than one workgroup of columns, whole row tiles
])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("scale", [1.0, 100.0])
def test_backward_without_a_cache(rb, d, V, prompts, length, layout, scale):
    """Backward without a cache, all rows in one chunk or (smallest workspace) in chunks of 256: the oracle's bounds, and in
    every chunk as close to it as with the packed copies of W (tuning key 2 = 8); scale: logits hundreds of nats apart."""
    print(f"no cache d {d} V {V} {layout} scale {scale}", flush=True)
    spec = wl.small_spec("no_cache", "bf16", d=d, V=V, prompts=prompts, G=4, len_lo=length - 9, len_hi=length, reward="uniform")
    w, g = _make(spec)
    W = (w["W"].float() * scale).to(torch.bfloat16)
    Wg = (W if layout == "dv" else W.t().contiguous()).cuda()
    lay = rb.W_DV if layout == "dv" else rb.W_VD
    H, _, _, mask = _oracle_inputs(w)
    # any token but the likeliest: where that one's probability is 1 to fp32, 1 - p has no correct digits to compare
    other = torch.randint(1, V, tuple(w["tokens"].shape), generator=torch.Generator().manual_seed(3))
    w["tokens"] = ((torch.from_numpy(H @ _np(W)).argmax(-1) + other) % V).to(torch.int32)
    g["tokens"], tok = w["tokens"].cuda(), _np(w["tokens"])
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], Wg, g["tokens"], g["mask"], w_layout=lay)
    ref = orc.iw_pg_loss_fwd_bwd(H, _np(W), tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"])
    far = {}
    try:
        for packed, min_ws in ((False, False), (False, True), (True, False)):
            rb.rapid_set_tuning(2, 8 if packed else 0)
            buf = rb.IwPgBuffers(g["hidden"], Wg, w["K"], lay, minimum_workspace=min_ws)
            out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], Wg, g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"],
                                              w["K"], buffers=buf, w_layout=lay)
            torch.cuda.synchronize()
            dW = _np(out.dW) if layout == "dv" else _np(out.dW).T
            assert out.dev_status.item() == 0
            _dh_ok(out.dhidden, ref["dH"])
            _dw_ok(dW, ref["dW"])
            far[packed, min_ws] = _rel(dW, ref["dW"]), _rel(_np(out.dhidden), ref["dH"])
    finally:
        rb.rapid_set_tuning(2, 0)
    print("relative errors (dW, dHidden): " + str(far), flush=True)
    for in_place in ((False, False), (False, True)):
        # the same products summed in another order, which moves some of the roundings of dz and dHidden to bf16
        assert all(a <= b * 1.02 for a, b in zip(far[in_place], far[True, False]))


@pytest.mark.parametrize("d", [256, 448])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("cache", [False, True])
def test_nan_weight_is_not_hidden(rb, d, layout, cache):
    """One weight that is not a number: the vocabulary column's gradient and every token's dHidden are not numbers either."""
    print(f"NaN weight d {d} {layout} cache {cache}", flush=True)
    w, g = _make(wl.small_spec("nan", "bf16", d=d, V=600, prompts=4, G=4, len_lo=20, len_hi=30, reward="uniform"))
    g["tokens"][g["tokens"] == 333] = 7     # the log-probs themselves stay finite: the column's slot drops out of the sum
    W = g["W"].clone()
    W[5, 333] = float("nan")
    W, lay = (W, rb.W_DV) if layout == "dv" else (W.t().contiguous(), rb.W_VD)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], W, g["tokens"], g["mask"], None, g["rewards"], g["group_ids"], w["K"],
                                      w_layout=lay, logits_cache=cache)
    torch.cuda.synchronize()
    dW = out.dW if layout == "dv" else out.dW.t()
    assert dW[:, 333].isnan().all()
    assert out.dhidden[g["mask"] != 0].isnan().all() and (out.dhidden[g["mask"] == 0] == 0).all()


@pytest.mark.parametrize("d", [136, 192, 200, 384, 448, 568])     # tiles of 192 (one, whole, two, three) and of 224
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("packed", [False, True])
def test_hidden_tiles_of_192_and_224(rb, d, layout, packed):
    """dHidden in tiles of the hidden dimension that are no power of two, with few tiles (cut): the head packed, in a batch
    padded to more positions than it is read in place for; read in place (short contractions: tiles of 128 instead)."""
    print(f"hidden tiles d {d} {layout} packed {packed}", flush=True)
    spec = wl.small_spec("tiles", "bf16", d=d, V=520, prompts=8, G=5, len_lo=10, len_hi=420 if packed else 40, reward="uniform")
    for cache in (False, True):
        w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache)
        _check_pair(rb, spec, out, ref, layout)


# Past the bounds of the tiles of 128 x 128: more than 4096 row tiles x K steps for dHidden (9 row tiles of positions, few
# of them tokens; the head read in place), more than 128 tiles for dW.
@pytest.mark.parametrize("d,V", [
    (128, 33000), (256, 33000),     # tiles of 128 and of 256
    (136, 33000), (192, 33000),     # one tile of 192, ragged and whole
    (576, 11104),                   # three of 192
    (200, 33000), (448, 16704),     # dHidden one and two tiles of 224, dW of 256
])
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_hidden_tiles_of_long_contractions(rb, d, V, layout):
    cache = layout == "vd"
    print(f"hidden tiles, long contractions d {d} V {V} {layout}", flush=True)
    spec = wl.small_spec("long", "bf16", d=d, V=V, prompts=3, G=3, len_lo=8, len_hi=256, reward="uniform")
    assert -(-d // 256) * 9 * -(-V // 64) > 4096 and -(-d // 256) * -(-V // 256) > 128
    w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache)
    _check_pair(rb, spec, out, ref, layout)
    _dw_in_every_form(rb, w, layout, cache)


@pytest.mark.parametrize("rows", [1, 64, 65, 192, 193, 257, 300, 1030])    # tokens of the last row tile: one to all waves' shares
@pytest.mark.parametrize("V", [700, 33330, 67000])                        # less than one round of workgroups, and up to nine
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_forward_with_a_short_last_row_tile(rb, rows, V, layout):
    print(f"short last row tile rows {rows} V {V} {layout}", flush=True)
    gen = torch.Generator().manual_seed(rows)
    hidden = torch.randn((1, rows, 72), generator=gen).to(torch.bfloat16)
    W = (torch.randn((72, V), generator=gen) * 0.3).to(torch.bfloat16)
    tokens = torch.randint(0, V, (1, rows), generator=gen, dtype=torch.int32)
    z = hidden[0].double() @ W.double()
    lse = torch.logsumexp(z, -1)
    want = z.gather(1, tokens[0].long()[:, None])[:, 0] - lse
    logp, got = rb.rapid_logprob_fwd(hidden.cuda(), (W if layout == "dv" else W.t().contiguous()).cuda(), tokens.cuda(),
                                     torch.ones((1, rows), dtype=torch.uint8).cuda(), want_lse=True,
                                     w_layout=rb.W_DV if layout == "dv" else rb.W_VD)
    torch.cuda.synchronize()
    # fp32 sums of 72 products of magnitude up to about 4, and of the exponentials
    assert (logp.cpu().double()[0] - want).abs().max() <= 2e-5 and (got.cpu().double()[0] - lse).abs().max() <= 2e-5


@pytest.mark.parametrize("d,V,prompts,length", [
    (8, 9, 1, 2),            # one tile of 128, one step
    (128, 1024, 2, 64),      # whole tiles of 128
    (136, 1032, 3, 90),      # two of the hidden dimension, remainders in every direction
    (584, 264, 4, 50),       # Hc padded to tiles of 192, read in tiles of 128
    (256, 4096, 8, 100),     # more K steps than segments
])
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("cache", [False, True])
def test_short_contractions_in_tiles_of_128(rb, d, V, prompts, length, layout, cache):
    print(f"tiles of 128 d {d} V {V} rows {prompts * 4 * length} {layout} cache {cache}", flush=True)
    spec = wl.small_spec("short", "bf16", d=d, V=V, prompts=prompts, G=4, len_lo=max(1, length - 9), len_hi=length, reward="uniform")
    w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache)
    _check_pair(rb, spec, out, ref, layout)


@pytest.mark.parametrize("d,min_ws", [(64, False), (448, True)])
@pytest.mark.parametrize("cache", [False, True])
def test_idle_generations_with_large_logits(rb, d, min_ws, cache):
    """Generations without gradient fill the last row tile up behind those that have one: exp of their logits, which
    overflows here, must not reach dW."""
    print(f"idle generations with large logits d {d} min_ws {min_ws} cache {cache}", flush=True)
    w, g = _make(wl.small_spec("idle", "bf16", d=d, V=300, prompts=6, G=4, len_lo=12, len_hi=18, reward="uniform"))
    idle = w["group_ids"] == 2
    w["rewards"][idle] = 0.0
    w["hidden"][idle] *= 4000.0
    live_rows = int(w["mask"][~idle].sum())
    assert live_rows % 256 and live_rows > 256
    g = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in w.items()}
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W"], g["tokens"], g["mask"])
    H, W, tok, mask = _oracle_inputs(w)
    assert (H[_np(idle.float()) != 0] @ W).max() > 200
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"])
    buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=cache, minimum_workspace=min_ws)
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"],
                                      w["K"], buffers=buf, logits_cache=cache)
    torch.cuda.synchronize()
    assert out.dev_status.item() == 0
    _dh_ok(out.dhidden, ref["dH"])
    _dw_ok(out.dW, ref["dW"])


@pytest.mark.parametrize("waves", [4, 16])
def test_short_last_row_tile_in_other_geometries(rb, waves):
    """A last row tile of 40 tokens behind a whole one whose rows 64 to 127 have logits in the hundreds, several tiles per
    workgroup: what the cache holds for rows past the last token is formed from rows of zeros whatever the geometry."""
    print(f"short last row tile, {waves} waves", flush=True)
    gen = torch.Generator().manual_seed(1)
    N, T, d, V = 4, 74, 128, 70000
    hidden = torch.randn((N * T, d), generator=gen)
    hidden[64:128] *= 400.0
    hidden = hidden.view(N, T, d).to(torch.bfloat16).cuda()
    W = (torch.randn((d, V), generator=gen) * 0.02).to(torch.bfloat16).cuda()
    tokens = torch.randint(0, V, (N, T), generator=gen, dtype=torch.int32).cuda()
    mask = torch.ones((N, T), dtype=torch.uint8).cuda()
    logp_b, _ = rb.rapid_logprob_fwd(hidden, W, tokens, mask)
    rewards, group = torch.tensor([1.0, 0.0, 0.5, 0.0]).cuda(), torch.zeros(N, dtype=torch.int32).cuda()
    got = {}
    try:
        for w in (8, waves):
            rb.rapid_set_tuning(2, w)
            out = rb.rapid_iw_pg_loss_fwd_bwd(hidden, W, tokens, mask, logp_b, rewards, group, 1, logits_cache=True)
            torch.cuda.synchronize()
            assert out.dev_status.item() == 0
            got[w] = _np(out.dW)
    finally:
        rb.rapid_set_tuning(2, 0)
    assert np.isfinite(got[waves]).all()
    assert _rel(got[waves], got[8]) <= 1e-5         # the same bf16 operands, fp32 sums of 296 terms in another order


@pytest.mark.parametrize("V", [8, 256, 257, 2048, 2049, 16384, 16385])     # 2 slots per 256 entries: 1, 4 or 16 waves fold them
@pytest.mark.parametrize("rows", [1, 32, 77])
def test_log_sum_exp_over_few_and_many_slots(rb, V, rows):
    print(f"log-sum-exp V {V} rows {rows}", flush=True)
    gen = torch.Generator().manual_seed(V + rows)
    hidden = torch.randn((1, rows, 64), generator=gen).to(torch.bfloat16)
    W = (torch.randn((64, V), generator=gen) * 0.5).to(torch.bfloat16)
    tokens = torch.randint(0, V, (1, rows), generator=gen, dtype=torch.int32)
    z = hidden[0].double() @ W.double()
    lse = torch.logsumexp(z, -1)
    want = z.gather(1, tokens[0].long()[:, None])[:, 0] - lse
    logp, got = rb.rapid_logprob_fwd(hidden.cuda(), W.cuda(), tokens.cuda(), torch.ones((1, rows), dtype=torch.uint8).cuda(), want_lse=True)
    torch.cuda.synchronize()
    # fp32 sums of 64 products of magnitude up to about 6, and of the exponentials
    assert (logp.cpu().double()[0] - want).abs().max() <= 2e-5 and (got.cpu().double()[0] - lse).abs().max() <= 2e-5


@pytest.mark.parametrize("N,T", [(2, 511), (3, 512), (2, 513), (2, 767), (5, 1028), (3, 4095), (2, 4096), (1, 8197)])   # 1, 2, .. 16 waves
@pytest.mark.parametrize("p", [0.5, 1.0])
def test_long_sequences_are_compacted_by_several_waves(rb, N, T, p):
    print(f"several waves N {N} T {T} p {p}", flush=True)
    gen = torch.Generator().manual_seed(N * T)
    mask = (torch.rand((N, T), generator=gen) < p).to(torch.uint8)
    mask[:, -1] = 1
    seq_len, cu, row_index = rb.rapid_compaction(mask.cuda())
    o_len, o_cu, o_rows = orc.compaction(_np(mask))
    assert np.array_equal(_np(seq_len), o_len) and np.array_equal(_np(cu), o_cu) and np.array_equal(_np(row_index)[:o_cu[-1]], o_rows)
    hidden = torch.randn((N, T, 8), generator=gen).to(torch.bfloat16)
    W = torch.randn((8, 24), generator=gen).to(torch.bfloat16)
    tokens = torch.randint(0, 24, (N, T), generator=gen, dtype=torch.int32)
    want = torch.log_softmax(hidden.double() @ W.double(), -1).gather(2, tokens.long()[:, :, None])[:, :, 0] * mask
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    logp, _ = rb.rapid_logprob_fwd(hidden.cuda(), W.cuda(), tokens.cuda(), mask.cuda(), dev_status=status)
    torch.cuda.synchronize()
    assert status.item() == 0
    # fp32 sums of 8 products of magnitude up to about 16
    assert (logp.cpu().double() - want).abs().max() <= 2e-5 and (logp.cpu()[mask == 0] == 0).all()
    tokens[-1, -1] = 24
    rb.rapid_logprob_fwd(hidden.cuda(), W.cuda(), tokens.cuda(), mask.cuda(), dev_status=status)
    torch.cuda.synchronize()
    assert status.item() == rb.STATUS_BAD_TOKEN


@pytest.mark.parametrize("N,K", [(1, 1), (64, 3), (255, 1), (257, 5), (1025, 300)])     # one block of checks and several, a last short one
def test_generations_without_a_group(rb, N, K):
    """Group ids out of range at both ends of the batch and in between: advantage 0, their own weight, the status bits."""
    print(f"generations without a group N {N} K {K}", flush=True)
    rng = np.random.default_rng(N)
    R, s = rng.random(N).astype(np.float32), rng.normal(size=N).astype(np.float32)
    gid = rng.integers(0, K, size=N).astype(np.int32)
    lost = np.unique([0, N // 2, N - 1])
    gid[lost] = [-1, K, K + 7][:len(lost)]
    keep = np.setdiff1d(np.arange(N), lost)
    status = torch.zeros(1, dtype=torch.int32).cuda()
    out = rb.rapid_group_advantage(torch.from_numpy(R).cuda(), torch.from_numpy(gid).cuda(), K, seq_logratio=torch.from_numpy(s).cuda(),
                                   eta=2.0, dev_status=status)
    torch.cuda.synchronize()
    ref = orc.group_advantage(R[keep], gid[keep], K, s=s[keep], eta=2.0)
    assert status.item() == rb.STATUS_BAD_GROUP
    assert np.array_equal(_np(out["group_size"]), ref["group_size"])
    assert (_np(out["adv"])[lost] == 0.0).all() and np.allclose(_np(out["adv"])[keep], ref["adv"], atol=2e-6)
    assert np.allclose(_np(out["weight"]), orc.clipped_weight(s.astype(np.float64), 2.0), rtol=1e-6)


@pytest.mark.parametrize("d", [640, 1040])      # their fastest tiles pad further than the smallest workspace has room for
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("cache", [False, True])
def test_smallest_workspace_has_room_for_other_tiles_only(rb, d, layout, cache):
    print(f"smallest workspace d {d} {layout} cache {cache}", flush=True)
    spec = wl.small_spec("min_ws", "bf16", d=d, V=1500, prompts=6, G=4, len_lo=20, len_hi=60, reward="uniform")
    w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=cache, min_ws=True)
    _check_pair(rb, spec, out, ref, layout)


@pytest.mark.parametrize("prompts,G,length", [
    (256, 4, 16),      # 1024 generations, 16384 positions: the most whose lengths and plan one block makes in the LDS
    (256, 4, 15),      # the same with odd rows
    (256, 4, 17),      # lengths counted in a launch of their own, plan in the LDS
    (256, 4, 32),      # 32768 positions: the most of which a wave packs one
    (256, 4, 33),      # more than one position per wave, odd rows
    (257, 4, 9),       # plan in memory
    (1, 3, 1),         # one position each
    (2, 3, 130), (3, 5, 258), (1, 2, 519),     # 8 to 64 lanes per generation, rows that are no whole words
])
@pytest.mark.parametrize("mode", ["recompute", "cache", "chunks", "f32"])
def test_plan_and_rows_of_a_batch(rb, prompts, G, length, mode):
    print(f"plan and rows {prompts} x {G} x {length} {mode}", flush=True)
    dtype = "f32" if mode == "f32" else "bf16"
    spec = wl.small_spec("rows", dtype, d=24, V=40, prompts=prompts, G=G, len_lo=max(1, length // 3), len_hi=length)
    kw = dict(recompute={}, cache=dict(logits_cache=True), chunks=dict(logits_cache=True), f32={})[mode]
    w, out, ref = _run_pair(rb, spec, min_ws=mode == "chunks" and G * length <= 256, **kw)
    _check_pair(rb, spec, out, ref)


@pytest.mark.parametrize("prompts,G,length", [
    (7, 5, 40),       # the estimator in one block, teams of 8 lanes
    (3, 17, 130),     # teams of 32 lanes, groups of more than 16
    (1, 2, 1030),     # two waves per generation and more
    (2, 3, 1500),     # 9000 positions: the log ratios in a launch of their own, by several waves each
    (70, 4, 33),      # 9240 positions of short generations
])
@pytest.mark.parametrize("kw", [
    dict(baseline_mode=2, coef_mode=1, eta=1.05), dict(baseline_mode=1, normalized_grads=True), dict(ratio_level=1, eta=1.1),
    dict(ratio_level=1, normalized_grads=True, coef_mode=1),
])
@pytest.mark.parametrize("scattered", [False, True])
def test_estimator_of_a_small_batch(rb, prompts, G, length, kw, scattered):
    print(f"estimator {prompts} x {G} x {length} {kw} scattered {scattered}", flush=True)
    spec = wl.small_spec("estimator", "bf16", d=24, V=40, prompts=prompts, G=G, len_lo=max(1, length // 2), len_hi=length, reward="uniform")
    w, g = _make(spec)
    gid = w["group_ids"]
    if scattered:
        gid = gid[torch.randperm(gid.numel(), generator=torch.Generator().manual_seed(1))].contiguous()
    H, W, tok, mask = _oracle_inputs(w)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], gid.cuda(), w["K"], **kw)
    torch.cuda.synchronize()
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(gid), w["K"], **kw)
    ref["slack"] = pb.coefficient_slack(ref, _np(w["rewards"]), mask)
    _check_pair(rb, spec, out, ref)
    # the same call's outputs from the stand-alone entry points
    s, tl = rb.rapid_seq_logratio(out.logp_cur, logp_b, g["mask"], want_tokens=True)
    assert torch.equal(tl, out.tok_logratio) and torch.allclose(s, out.seq_logratio, rtol=2.0 ** -23, atol=0)


# pieces of 128 generations listed by a wave each; from 4 waves to 16 in the block
@pytest.mark.parametrize("K,G,T", [(512, 2, 3), (2, 2, 3), (13, 5, 3), (43, 3, 20), (64, 2, 40), (3, 300, 8), (257, 3, 40), (1000, 1, 8)])
@pytest.mark.parametrize("kw", [dict(baseline_mode=2, eta=1.05), dict(ratio_level=1, normalized_grads=True)])
@pytest.mark.parametrize("faulty", [False, True])
def test_estimator_of_scattered_groups(rb, K, G, T, kw, faulty):
    """Groups whose members lie anywhere; "faulty": with group ids out of range, which are flagged and belong to no group (advantage
    0: a group of its own with reward 0 for the oracle), and a reward that is not finite, which counts as 0."""
    N = K * G
    print(f"scattered groups {K} x {G} x {T} {kw} faulty {faulty}", flush=True)
    spec = wl.small_spec("scattered", "bf16", d=24, V=40, prompts=K, G=G, len_lo=1, len_hi=T, reward="uniform")
    w, g = _make(spec)
    gid = np.random.default_rng(N).permutation(_np(w["group_ids"]).astype(np.int32))
    rewards = _np(w["rewards"]).astype(np.float32)
    ref_gid, ref_rewards, ref_K, bits = gid.copy(), rewards.copy(), K, 0
    if faulty and N >= 8:
        for i, (n, bad) in enumerate(zip(np.random.default_rng(7).choice(N, 3, replace=False), (-1, K, 2 ** 31 - 1))):
            gid[n], ref_gid[n], ref_rewards[n] = bad, K + i, 0.0
        odd = int(np.flatnonzero((gid >= 0) & (gid < K))[N // 3])
        rewards[odd] = np.inf
        ref_rewards[odd] = 0.0
        ref_K, bits = K + 3, rb.STATUS_BAD_GROUP | rb.STATUS_NONFINITE_REWARD
    H, W, tok, mask = _oracle_inputs(w)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, torch.from_numpy(rewards).cuda(),
                                      torch.from_numpy(gid).cuda(), K, **kw)
    torch.cuda.synchronize()
    assert out.dev_status.item() == bits
    out.dev_status.zero_()
    ref = orc.iw_pg_loss_fwd_bwd(H, W, tok, mask, _np(logp_b), ref_rewards, ref_gid, ref_K, **kw)
    ref["slack"] = pb.coefficient_slack(ref, ref_rewards, mask)
    _check_pair(rb, spec, out, ref)


def test_estimator_time_of_scattered_groups(rb):
    """512 pairs among 1024 generations take about as long scattered as side by side (1.9 times as long while a team of lanes looked
    through the batch for every group)."""
    N, T = 1024, 8
    gen = torch.Generator(device="cuda").manual_seed(5)
    hidden = torch.randn((N, T, 16), generator=gen, device="cuda")
    W = torch.randn((16, 40), generator=gen, device="cuda")
    tokens = torch.randint(0, 40, (N, T), generator=gen, device="cuda", dtype=torch.int32)
    mask = torch.ones((N, T), dtype=torch.uint8, device="cuda")
    lp, _ = rb.rapid_logprob_fwd(hidden, W, tokens, mask)
    rewards = torch.rand(N, generator=gen, device="cuda")
    buf = rb.IwPgBuffers(hidden, W, N // 2)

    def microseconds(gid):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                rb.rapid_iw_pg_loss_fwd_bwd(hidden, W, tokens, mask, lp, rewards, gid, N // 2, buffers=buf)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 10 * 1e3)
        return min(times)
    adjacent = (torch.arange(N, device="cuda") // 2).to(torch.int32)
    side_by_side = microseconds(adjacent)
    scattered = microseconds(adjacent[torch.randperm(N, generator=gen, device="cuda")].contiguous())
    print(f"step of 512 pairs: side by side {side_by_side:.0f} us, scattered {scattered:.0f} us", flush=True)
    assert scattered <= 1.4 * side_by_side


@pytest.mark.parametrize("d", [8, 512, 520, 1032, 1544, 2048, 2056])      # 1 to 4 chunks of 16 bytes per lane, and wider rows
@pytest.mark.parametrize("mode", ["recompute", "chunks"])
def test_final_norm_backward_by_width(rb, d, mode):
    print(f"final norm d {d} {mode}", flush=True)
    spec = wl.small_spec("norm", "bf16", d=d, V=72, prompts=5, G=3, len_lo=9, len_hi=40, reward="uniform")
    w, g = _make(spec)
    gen = torch.Generator().manual_seed(d)
    x = (g["hidden"].cpu().float() * torch.exp(torch.randn((*g["hidden"].shape[:2], 1), generator=gen))).to(torch.bfloat16).cuda()
    wgt = (1.0 + 0.3 * torch.randn(d, generator=gen)).to(torch.bfloat16).cuda()
    logp_b, _ = rb.rapid_logprob_fwd(x, g["W_old"], g["tokens"], g["mask"], rms_weight=wgt)
    buf = rb.IwPgBuffers(x, g["W"], w["K"], minimum_workspace=mode == "chunks", logits_cache=mode == "chunks")
    out = rb.rapid_iw_pg_loss_fwd_bwd(x, g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], w["K"],
                                      buffers=buf, logits_cache=mode == "chunks", rms_weight=wgt)
    torch.cuda.synchronize()
    _, W, tok, mask = _oracle_inputs(w)
    ref = orc.iw_pg_loss_fwd_bwd(_np(x), W, tok, mask, _np(logp_b), _np(w["rewards"]), _np(w["group_ids"]), w["K"],
                                 rms_weight=_np(wgt), rms_eps=1e-6, round_normed_hidden=True)
    assert out.dev_status.item() == 0
    # as test_fwd_bwd_with_final_rmsnorm: dL/dx is formed from a dL/dh that is rounded to bf16 first
    assert _rel(_np(out.dhidden), ref["dH"]) <= 2e-2 and _rel(_np(out.dW), ref["dW"]) <= 2e-2
    assert _rel(_np(out.drms_weight), ref["d_rms_weight"]) <= 2e-2
    assert np.abs(_np(out.drms_weight) - ref["d_rms_weight"]).max() <= 2.0 ** -6 * np.abs(ref["d_rms_weight"]).max()


@pytest.mark.parametrize("d", [2048, 2056])       # one pass over a row, and two
def test_final_norm_backward_of_more_regions_than_the_partial_sums_have_room_for(rb, d):
    """The smallest cache makes thousands of regions of 256 rows of a large batch, whose partial sums of dL/dweight (a row each) are
    more than the 128 MiB they lie in otherwise.  Few positions hold tokens: the same tokens as a batch of their own, without a
    cache, give the same gradients."""
    N, T, V, K, length = 8193, 256, 131072, 8193, 1
    print(f"final norm in {2 * N + 1} regions, d {d}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(2)
    small = torch.randn((N, length, d), generator=gen, device="cuda").to(torch.bfloat16)
    W = (torch.randn((d, V), generator=gen, device="cuda") * d ** -0.5).to(torch.bfloat16)
    wgt = (1.0 + 0.3 * torch.randn(d, generator=gen, device="cuda")).to(torch.bfloat16)
    tokens = torch.randint(0, V, (N, length), generator=gen, device="cuda", dtype=torch.int32)
    ones = torch.ones((N, length), dtype=torch.uint8, device="cuda")
    rewards = torch.rand(N, generator=gen, device="cuda")
    gid = torch.arange(N, device="cuda", dtype=torch.int32)
    coef = ((rewards - 0.5) / N).contiguous()
    wide = lambda t: torch.cat([t, torch.zeros((N, T - length, *t.shape[2:]), dtype=t.dtype, device="cuda")], 1)
    hidden, mask = wide(small), wide(ones)
    nbytes = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, V, K, rb.DTYPE_BF16, minimum=True)
    assert rb.rapid_logits_cache_rows(N, T, d, V, K, 0, nbytes) == 256
    assert (2 * (N * T // 256) + 1) * d * 4 > 128 << 20
    buf = rb.IwPgBuffers(hidden, W, K, workspace_bytes=nbytes)
    got = rb.rapid_iw_pg_loss_fwd_bwd(hidden, W, wide(tokens), mask, None, rewards, gid, K, buffers=buf, logits_cache=True,
                                      coef_override=coef, rms_weight=wgt)
    torch.cuda.synchronize()
    assert got.dev_status.item() == 0 and got.read_diag()["n_tokens"] == N * length
    want = rb.rapid_iw_pg_loss_fwd_bwd(small, W, tokens, ones, None, rewards, gid, K, coef_override=coef, rms_weight=wgt)
    torch.cuda.synchronize()
    assert torch.equal(got.logp_cur[:, :length], want.logp_cur)
    # two backward modes: dL/dh of both is rounded to bf16 from sums taken in another order
    assert _rel(_np(got.drms_weight), _np(want.drms_weight)) <= 4e-3
    assert _rel(_np(got.dhidden[:, :length]), _np(want.dhidden)) <= 4e-3
    assert not got.dhidden[:, length:].any()


@pytest.mark.parametrize("N,T", [(1, 1), (3, 5), (7, 33), (1, 4096), (1, 4097), (2, 4096), (64, 128), (73, 113)])   # up to 8192 positions, T <= 4096: no plan
@pytest.mark.parametrize("dtype,layout", [("bf16", "dv"), ("bf16", "vd"), ("f32", "dv")])
def test_rows_without_a_plan(rb, N, T, dtype, layout):
    print(f"rows without a plan {N} x {T} {dtype} {layout}", flush=True)
    gen = torch.Generator().manual_seed(N * T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    mask = (torch.rand((N, T), generator=gen) < 0.6).to(torch.uint8)
    hidden = torch.randn((N, T, 24), generator=gen).to(dt)
    W = (torch.randn((24, 40), generator=gen) * 0.3).to(dt)
    tokens = torch.randint(0, 40, (N, T), generator=gen, dtype=torch.int32)
    z = hidden.double() @ W.double()
    lse = torch.logsumexp(z, -1)
    want = (z.gather(2, tokens.long()[:, :, None])[:, :, 0] - lse) * mask
    Wg = (W if layout == "dv" else W.t().contiguous()).cuda()
    for at in (0, 1, 4):            # the mask's alignment decides how it is read
        buf = torch.zeros(N * T + 16, dtype=torch.uint8, device="cuda")
        m = buf[at:at + N * T].view(N, T)
        m.copy_(mask)
        logp, got = rb.rapid_logprob_fwd(hidden.cuda(), Wg, tokens.cuda(), m, w_layout=rb.W_DV if layout == "dv" else rb.W_VD, want_lse=True)
        torch.cuda.synchronize()
        # fp32 sums of 24 products (bf16 path) and of 40 exponentials
        assert (logp.cpu().double() - want).abs().max() <= 2e-5 and (got.cpu().double() - lse * mask).abs().max() <= 2e-5


# more than 8192 positions and no gradient rows: an index in front of the rows; one wave per generation and (from 512 positions on) several
@pytest.mark.parametrize("N,T", [(4100, 2), (130, 64), (33, 249), (17, 511), (16, 513), (9, 1024), (3, 2731), (3, 4096)])
@pytest.mark.parametrize("dtype,layout", [("bf16", "dv"), ("bf16", "vd"), ("f32", "dv")])
def test_rows_with_an_index(rb, N, T, dtype, layout):
    print(f"rows with an index {N} x {T} {dtype} {layout}", flush=True)
    gen = torch.Generator().manual_seed(N * T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    mask = (torch.rand((N, T), generator=gen) < 0.6).to(torch.uint8)
    hidden = torch.randn((N, T, 24), generator=gen).to(dt)
    W = (torch.randn((24, 40), generator=gen) * 0.3).to(dt)
    tokens = torch.randint(0, 40, (N, T), generator=gen, dtype=torch.int32)
    z = hidden.double() @ W.double()
    lse = torch.logsumexp(z, -1)
    want = (z.gather(2, tokens.long()[:, :, None])[:, :, 0] - lse) * mask
    Wg = (W if layout == "dv" else W.t().contiguous()).cuda()
    for at in (0, 1, 4):            # the mask's alignment decides how it is read
        buf = torch.zeros(N * T + 16, dtype=torch.uint8, device="cuda")
        m = buf[at:at + N * T].view(N, T)
        m.copy_(mask)
        logp, got = rb.rapid_logprob_fwd(hidden.cuda(), Wg, tokens.cuda(), m, w_layout=rb.W_DV if layout == "dv" else rb.W_VD, want_lse=True)
        sl, cu, ri = rb.rapid_compaction(m)
        torch.cuda.synchronize()
        # as test_rows_without_a_plan: fp32 sums of 24 products (bf16 path) and of 40 exponentials
        assert (logp.cpu().double() - want).abs().max() <= 2e-5 and (got.cpu().double() - lse * mask).abs().max() <= 2e-5
        count = int(mask.sum())
        assert torch.equal(sl.cpu().long(), mask.long().sum(1)) and int(cu[N]) == count
        assert torch.equal(ri.cpu()[:count].long(), torch.nonzero(mask.flatten()).flatten()) and bool((ri[count:] == -1).all())


@pytest.mark.parametrize("N,T", [(3, 37), (2, 300), (2, 1027)])
def test_rows_by_position_wherever_the_mask_starts(rb, N, T):
    """Every distance of the mask from a 16-byte boundary, counted up to every position: the same rows, the same bits."""
    print(f"mask alignment {N} x {T}", flush=True)
    gen = torch.Generator().manual_seed(T)
    mask = (torch.rand((N, T), generator=gen) < 0.6).to(torch.uint8)
    hidden = torch.randn((N, T, 8), generator=gen).to(torch.bfloat16).cuda()
    W = torch.randn((8, 8), generator=gen).to(torch.bfloat16).cuda()
    tokens = torch.randint(0, 8, (N, T), generator=gen, dtype=torch.int32).cuda()
    every, _ = rb.rapid_logprob_fwd(hidden, W, tokens, torch.ones((N, T), dtype=torch.uint8, device="cuda"))
    rows = torch.nonzero(mask.flatten()).flatten()
    for at in range(16):
        buf = torch.ones(N * T + 32, dtype=torch.uint8, device="cuda")      # ones around the mask: nothing of them may be counted
        m = buf[at:at + N * T].view(N, T)
        m.copy_(mask)
        logp, _ = rb.rapid_logprob_fwd(hidden, W, tokens, m)
        _, _, index = rb.rapid_compaction(m)
        torch.cuda.synchronize()
        assert torch.equal(logp, every * m) and torch.equal(index.cpu()[:len(rows)].long(), rows)


def test_compaction_time_is_that_of_the_positions(rb):
    """The same two million positions in 256 long and in 4096 short generations: with a wave for every 16 positions, each counting
    its generation up to there, the short ones took six times as long."""
    def microseconds(N, T):
        mask = torch.ones((N, T), dtype=torch.uint8, device="cuda")
        rb.rapid_compaction(mask)
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                rb.rapid_compaction(mask)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) / 20 * 1e3)
        return min(times)
    long, short = microseconds(256, 8192), microseconds(4096, 512)
    print(f"compaction: 256 x 8192 {long:.1f} us, 4096 x 512 {short:.1f} us", flush=True)
    assert short <= 3.0 * long + 20.0


@pytest.mark.parametrize("prompts,V", [(3, 1000), (40, 20000)])       # dHidden and dW in one launch, and in two
@pytest.mark.parametrize("cache", [False, True])
def test_stage_times_cover_dhidden_and_dw(rb, prompts, V, cache):
    print(f"stage times {prompts} prompts, V {V}, cache {cache}", flush=True)
    spec = wl.small_spec("stages", "bf16", d=256, V=V, prompts=prompts, G=4, len_lo=20, len_hi=60)
    w, g = _make(spec)
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    buf = rb.IwPgBuffers(g["hidden"], g["W"], w["K"], logits_cache=cache)
    try:
        rb.rapid_set_tuning(1, 1)
        for _ in range(3):
            rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, g["rewards"], g["group_ids"], w["K"],
                                        buffers=buf, logits_cache=cache)
        stages = rb.rapid_profile_read()
    finally:
        rb.rapid_set_tuning(1, 0)
    for name in ("compaction", "pack", "fwd_lse", "merge_lse", "estimator", "dz", "dh", "dw"):
        ms, spans = stages[name]
        assert spans % 3 == 0 and spans > 0 and ms > 0.0, (name, ms, spans)


def test_as_many_short_generations_as_before(rb):
    """2^24 + 5 generations of one position through the fp32 step: a launch of 2^32 threads is refused, so a generation's rows may
    not take a block of 256 threads."""
    N, K, d, V = 2 ** 24 + 5, 4, 8, 8
    print(f"{N} generations of one position", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    hidden = torch.randn((N, 1, d), generator=gen, device="cuda")
    W = torch.randn((d, V), generator=gen, device="cuda")
    tokens = torch.randint(0, V, (N, 1), generator=gen, device="cuda", dtype=torch.int32)
    mask = (torch.rand((N, 1), generator=gen, device="cuda") < 0.9).to(torch.uint8)
    rewards = torch.rand(N, generator=gen, device="cuda")
    gid = (torch.arange(N, device="cuda") * K // N).to(torch.int32)
    out = rb.rapid_iw_pg_loss_fwd_bwd(hidden, W, tokens, mask, None, rewards, gid, K)
    torch.cuda.synchronize()
    assert out.dev_status.item() == 0 and out.read_diag()["n_tokens"] == int(mask.sum())
    mean = torch.stack([rewards[gid == k].double().mean() for k in range(K)])
    for at in (slice(0, 4096), slice(N // 2, N // 2 + 4096), slice(N - 4096, N)):
        m = mask[at, 0].double()
        z = hidden[at, 0].double() @ W.double()
        logp = torch.log_softmax(z, -1)
        onehot = torch.nn.functional.one_hot(tokens[at, 0].long(), V).double()
        g = -(rewards[at].double() - mean[gid[at].long()]) / N
        dh = (g * m)[:, None] * ((onehot - logp.exp()) @ W.double().t())
        assert ((logp * onehot).sum(-1) * m - out.logp_cur[at, 0].double()).abs().max() <= 2e-6
        # the tolerances of the fp32 path
        assert (dh - out.dhidden[at, 0].double()).norm() <= 1e-5 * dh.norm()
        assert not out.dhidden[at, 0][m == 0].any()


@pytest.mark.parametrize("rows", [1, 7, 8, 9, 300, 1024, 1025])       # 8 columns per block up to 1024 rows, 32 above
def test_log_sum_exp_of_few_rows(rb, rows):
    """One order of summation whatever the launch: the rows of a short call have the bits of the same rows in a long one."""
    print(f"log-sum-exp of {rows} rows", flush=True)
    gen = torch.Generator().manual_seed(rows)
    hidden = torch.randn((1, 4097, 64), generator=gen).to(torch.bfloat16).cuda()
    W = (torch.randn((64, 16700), generator=gen) * 0.5).to(torch.bfloat16).cuda()
    tokens = torch.randint(0, 16700, (1, 4097), generator=gen, dtype=torch.int32).cuda()
    ones = torch.ones((1, 4097), dtype=torch.uint8).cuda()
    full, full_lse = rb.rapid_logprob_fwd(hidden, W, tokens, ones, want_lse=True)
    lp, lse = rb.rapid_logprob_fwd(hidden[:, :rows].contiguous(), W, tokens[:, :rows].contiguous(), ones[:, :rows].contiguous(), want_lse=True)
    assert torch.equal(lp, full[:, :rows]) and torch.equal(lse, full_lse[:, :rows])


@pytest.mark.parametrize("d", [448, 512, 1024, 1032])        # 7, 8, 16, 17 steps: W requested two steps ahead from 8 per row tile on
@pytest.mark.parametrize("rows", [5, 256, 257, 512, 513])
@pytest.mark.parametrize("layout", ["dv", "vd"])
def test_few_rows_request_w_two_steps_ahead(rb, d, rows, layout):
    """The same bits as from the packed copies (tuning key 2 = 8), plain and storing forward."""
    print(f"W two steps ahead d {d} rows {rows} {layout}", flush=True)
    spec = wl.small_spec("deep", "bf16", d=d, V=33000, prompts=1, G=1, len_lo=rows, len_hi=rows)
    w, g = _make(spec)
    W, lay = (g["W"], rb.W_DV) if layout == "dv" else (g["W"].t().contiguous(), rb.W_VD)
    got = []
    try:
        for waves in (0, 8):
            rb.rapid_set_tuning(2, waves)
            lp, _ = rb.rapid_logprob_fwd(g["hidden"], W, g["tokens"], g["mask"], w_layout=lay)
            out = rb.rapid_iw_pg_loss_fwd_bwd(g["hidden"], W, g["tokens"], g["mask"], lp, torch.ones(1, device="cuda"), g["group_ids"], 1,
                                              w_layout=lay, logits_cache=True)
            torch.cuda.synchronize()
            assert out.dev_status.item() == 0 and torch.equal(out.logp_cur, lp)
            got.append((lp, out.dW.clone(), out.dhidden.clone()))
    finally:
        rb.rapid_set_tuning(2, 0)
    assert torch.equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1:], got[1][1:]):      # dHidden and dW sum in another order
        assert _rel(_np(a), _np(b)) <= 4e-3


@pytest.mark.parametrize("d,V", [(8, 9), (120, 1001), (192, 999), (328, 2047), (576, 1003), (1032, 259)])    # vocabularies that are not read in place
@pytest.mark.parametrize("layout", ["dv", "vd"])
@pytest.mark.parametrize("mode", ["recompute", "cache"])
def test_packed_heads_of_small_batches(rb, d, V, layout, mode):
    """Both packed copies in one pass, tiles of 128 for dHidden and of 256 x 128 for the logits: [d, V] with V % 8 != 0, and (as
    more than 131072 positions would) a [V, d] head through tuning key 2 = 8, whose log-probs have the same bits."""
    print(f"packed head d {d} V {V} {layout} {mode}", flush=True)
    spec = wl.small_spec("packed", "bf16", d=d, V=V, prompts=5, G=3, len_lo=5, len_hi=40, reward="uniform")
    got = []
    try:
        for waves in (0, 8):
            rb.rapid_set_tuning(2, waves)
            w, out, ref = _run_pair(rb, spec, layout=layout, logits_cache=mode == "cache")
            _check_pair(rb, spec, out, ref, layout)
            got.append(out.logp_cur.clone())
    finally:
        rb.rapid_set_tuning(2, 0)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("V", [1, 255, 257, 1024, 1025, 2048, 2049, 4096, 4097])       # 4, 8, 16 logits per thread, and a loop
def test_fp32_log_sum_exp_by_vocabulary(rb, V):
    print(f"fp32 log-sum-exp V {V}", flush=True)
    gen = torch.Generator().manual_seed(V)
    hidden, W = torch.randn((3, 11, 20), generator=gen), torch.randn((20, V), generator=gen)
    tokens = torch.randint(0, V, (3, 11), generator=gen, dtype=torch.int32)
    z = hidden.double() @ W.double()
    lse = torch.logsumexp(z, -1)
    logp, got = rb.rapid_logprob_fwd(hidden.cuda(), W.cuda(), tokens.cuda(), torch.ones((3, 11), dtype=torch.uint8).cuda(), want_lse=True)
    torch.cuda.synchronize()
    want = z.gather(2, tokens.long()[:, :, None])[:, :, 0] - lse
    # logits of magnitude up to about 20 are stored as floats (2^-20 each), log-probs of up to 40 too
    assert (logp.cpu().double() - want).abs().max() <= 6e-6 and (got.cpu().double() - lse).abs().max() <= 4e-6


@pytest.mark.parametrize("T", [60, 4200])          # rows placed by position, and by row_index_kernel
@pytest.mark.parametrize("chunks", [False, True])
def test_generations_past_the_end_of_the_cache_place_no_rows(rb, T, chunks):
    """A broken opts.max_tokens: what the cache has room for is computed as ever, the other positions read 0 and nothing
    is written for them (a row of theirs would be another chunk's, or lie in front of or behind the buffers)."""
    print(f"past the end of the cache T {T} chunks {chunks}", flush=True)
    spec = wl.small_spec("past_end", "bf16", d=136, V=1100, prompts=20, G=3, len_lo=5, len_hi=60, sigma=0.02, reward="uniform")
    w, g = _make(spec, seed=4)
    N, T0, d = g["hidden"].shape
    pad = lambda t: torch.cat([t, torch.zeros((N, T - T0, *t.shape[2:]), dtype=t.dtype, device=t.device)], 1).contiguous()
    g = dict(g, **{k: pad(g[k]) for k in ("hidden", "tokens", "mask")})
    K, promise = w["K"], 512
    logp_b, _ = rb.rapid_logprob_fwd(g["hidden"], g["W_old"], g["tokens"], g["mask"])
    rewards = torch.ones_like(g["rewards"])
    args = (g["hidden"], g["W"], g["tokens"], g["mask"], logp_b, rewards, g["group_ids"], K)
    whole = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=rb.IwPgBuffers(g["hidden"], g["W"], K, logits_cache=True, max_tokens=4096),
                                        logits_cache=True, max_tokens=4096).logp_cur
    nbytes = rb.rapid_workspace_bytes(rb.OP_IW_PG_FWD_BWD_CACHED, N, T, d, spec.V, K, rb.DTYPE_BF16, max_tokens=promise)
    if chunks:
        nbytes -= 256
    Rcap = rb.rapid_logits_cache_rows(N, T, d, spec.V, K, promise, nbytes)
    assert Rcap == (256 if chunks else 512)
    per_group = g["mask"].long().sum(1).view(K, spec.G).sum(1).tolist()
    if chunks:                      # whole groups, in 2 * (512 / 256) + 1 chunks
        kept = rows = 0
        left = 2 * (promise // Rcap) + 1
        for n in per_group:
            if rows + n > Rcap:
                left, rows = left - 1, 0
                if left == 0:
                    break
            rows, kept = rows + n, kept + n
    else:
        kept = Rcap
    assert 0 < kept < sum(per_group)
    buf = rb.IwPgBuffers(g["hidden"], g["W"], K, workspace_bytes=nbytes)
    buf.logp_cur.fill_(float("nan"))
    out = rb.rapid_iw_pg_loss_fwd_bwd(*args, buffers=buf, logits_cache=True, max_tokens=promise)
    torch.cuda.synchronize()
    assert out.dev_status.item() & rb.STATUS_TOKEN_BOUND
    assert out.read_diag()["n_tokens"] == kept
    flat = g["mask"].flatten().bool()
    want = torch.where(flat & (flat.long().cumsum(0) <= kept), whole.flatten(), torch.zeros_like(whole.flatten()))
    assert torch.equal(out.logp_cur.flatten(), want)
