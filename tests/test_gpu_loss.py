"""GPU parity of nat_loss_fwd_bwd against the fp64 oracle (Eq. 1, 3, 5, 6/9; App. A).

Tolerances.  Per tensor, max-norm relative error ||gpu - oracle||_inf / ||oracle||_inf:
fp32 path <= 1e-5, bf16 path <= 2e-2 (dH, dW).  Because the one-hot term of dz dominates those
maxima when the soft-max is near-uniform, the two backward contractions are also checked on
their own at the same tolerance: rows of dW that no token targets against the largest such
entry, and dH with the one-hot term removed on both sides against the largest residual entry
(nat_testlib.contraction_errors; the rounding that the full value of an entry carries is allowed on
top, entry by entry: 2^-7 |dH| on the bf16 path, where the one-hot term is rounded to bf16 twice at a
unit roundoff of 2^-8 each, once as the patched numerator and once in the stored output; 2^-18 |dH| on
the fp32 path, whose sequential fp32 sum over V terms carries about sqrt(V) 2^-24 of the full value;
entries where the one-hot term is small are held to the bare tolerance).  Log-probs and the loss come from fp32 accumulators on both
paths and are held to an absolute 1e-4 (log-probs; 1e-5 relative on the fp32 path) and a
relative 1e-4 (loss; 1e-5 on the fp32 path).  Relative Frobenius errors are printed."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from nat_testlib import DEV, contraction_errors, hip_loss, make_loss_case, max_rel_err, oracle_loss, to_dev

TOL_F32 = 1e-5
TOL_BF16 = 2e-2
TOL_LOGP_ABS_BF16 = 1e-4          # fp32 accumulation of exact bf16 products; |logp| ~ 5..13
TOL_LOSS_BF16 = 1e-4


@pytest.fixture(scope="module")
def stage():
    from paper_2603_06619_amd.stage import LossStage
    return LossStage(DEV)


def check(out, ref, n, tol, case=None, logp_atol=None, label=None, all_zero=False):
    """Whole-tensor bounds, and (given the case's inputs) the contraction-only bounds.  all_zero: every advantage is 0."""
    bf16 = tol == TOL_BF16
    assert all_zero != bool(np.abs(ref["dH"]).max() > 0 and np.abs(ref["dW"]).max() > 0), "gradients of zero check nothing"
    tol_loss = TOL_LOSS_BF16 if bf16 else tol
    e_loss = abs(out["loss"].item() - ref["loss"]) / max(abs(ref["loss"]), 1e-300)
    assert e_loss <= tol_loss + 1e-12, ("loss", e_loss)
    logp = out["logp"].cpu().numpy()[:n].astype(np.float64)
    a_logp = float(np.abs(logp - ref["logp"]).max())
    if bf16:
        assert a_logp <= (TOL_LOGP_ABS_BF16 if logp_atol is None else logp_atol), ("logp abs", a_logp)
    e_logp = max_rel_err(logp, ref["logp"])
    dH = out["dH"].float().cpu().numpy()[:n]
    dW = out["dW"].cpu().numpy()
    e_dh = max_rel_err(dH, ref["dH"])
    e_dw = max_rel_err(dW, ref["dW"])
    assert e_logp <= (tol if not bf16 else 1e-4), ("logp", e_logp)
    assert e_dh <= tol, ("dH", e_dh)
    assert e_dw <= tol, ("dW", e_dw)
    if case is not None:
        ce = contraction_errors(dH, dW, ref, case["hidden"], case["W"], case["ids"], 2.0 ** -7 if bf16 else 2.0 ** -18)
        print("%s: loss %.1e logp abs %.1e | dH max %.1e fro %.1e residual %.1e (residual is %.1e of max) | "
              "dW max %.1e fro %.1e off-target rows %.1e (%.1e of max)"
              % (label or "case", e_loss, a_logp, e_dh, ce["dH_fro"], ce["dH_res"], ce["dH_res_share"], e_dw,
                 ce["dW_fro"], ce["dW_off"], ce["dW_off_share"]))
        assert ce["dH_res"] <= tol, ("dH without the one-hot term", ce)
        assert ce["dW_off"] <= tol, ("off-target rows of dW", ce)
    return e_logp, e_dh, e_dw


@pytest.mark.parametrize("n_tok,H,V", [(160, 64, 512), (1, 64, 512), (37, 48, 300), (300, 64, 512)])
def test_fp32_path(stage, n_tok, H, V):
    case = make_loss_case(10 + n_tok, n_tok, H, V, "f32", noise=0.15)
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "f32")
    check(out, ref, n_tok, TOL_F32, case)
    clipped = (ref["r"] > 1.2) | (ref["r"] < 0.8)
    assert n_tok < 30 or clipped.any()


@pytest.mark.parametrize("n_tok,H,V", [
    (33, 68, 1028),          # one past a 32-row tile on every axis, rows on 16 bytes
    (65, 31, 129),           # odd leading dimensions: no 16-byte operand reads
    (5, 7, 31),              # shorter than one step of one wavefront
    (31, 260, 2052),         # several 32-long steps per wavefront and a remainder
    (520, 64, 300),          # the dW contraction with more than one step per wavefront
])
def test_fp32_contraction_remainders(stage, n_tok, H, V):
    # tolerance: the path's 1e-5 (sums of at most 2052 fp32 products split over eight wavefronts stay below 1e-6)
    case = make_loss_case(40 + n_tok, n_tok, H, V, "f32", noise=0.15)
    ref = oracle_loss(**case)
    check(hip_loss(stage, case, "f32"), ref, n_tok, TOL_F32, case)


@pytest.mark.parametrize("V", [255, 256, 257, 512, 514, 1025, 2048, 2049, 4095, 4096, 4097])
def test_fp32_rows_kept_in_registers_and_read_again(stage, V):
    # up to 4096 logits of a token stay in registers, 1, 2, 4, 8 or 16 to a thread; an id outside the vocabulary among the tokens.  (Not V =
    # 513: in that draw the terms cancel to 1/670 of their sum, and a last place of the fp32 log-probs is 2.5e-4 of the loss)
    case = make_loss_case(1000 + V, 19, 48, V, "f32")
    check(hip_loss(stage, case, "f32"), oracle_loss(**case), 19, TOL_F32, case)
    ids = case["ids"].copy()
    ids[[0, 7]] = [V, -1]
    keep = np.delete(np.arange(19), [0, 7])
    out = hip_loss(stage, dict(case, ids=ids), "f32", want_entropy=True)
    part = {k: (v[keep] if k in ("hidden", "ids", "old_logp", "kept_seq", "kept_w") else v) for k, v in case.items()}
    ref = oracle_loss(**part)
    assert max_rel_err(out["dW"].cpu().numpy(), ref["dW"]) <= TOL_F32
    assert bool(torch.isnan(out["logp"][[0, 7]]).all()) and bool((out["dH"][[0, 7]] == 0).all())
    fwd = stage.logp(to_dev(case["hidden"]), to_dev(case["W"]), to_dev(ids), 19, want_entropy=True)
    assert torch.equal(fwd["logp"][keep], out["logp"][keep]) and torch.equal(fwd["entropy"][:19], out["entropy"][:19])


def test_fp32_vocabulary_beyond_the_columns_of_one_launch(stage):
    # the contractions take 2^20 columns of the logits to a launch.  (Whole tensors only: a wavefront's chain of 2^17 terms of dH
    # rounds by up to 2^17 x 2^-24 of the sum of their magnitudes, 8e-3 of the small part that check() takes alone)
    case = make_loss_case(9, 40, 4, (1 << 20) + 40, "f32", noise=0.15)
    case["ids"][:3] = [(1 << 20) - 1, 1 << 20, (1 << 20) + 39]
    check(hip_loss(stage, case, "f32"), oracle_loss(**case), 40, TOL_F32)


def test_fp32_chunked_workspace_and_accumulate(stage):
    import paper_2603_06619_amd as nat
    case = make_loss_case(5, 50, 64, 512, "f32")
    ref = oracle_loss(**case)
    small = nat.loss_workspace_min_bytes(50, 64, 512, nat.DTYPE_F32) + 6 * 512 * 4     # 7-token chunks
    out = hip_loss(stage, case, "f32", ws_bytes=small)
    check(out, ref, 50, TOL_F32, case)
    b0 = 2.0 ** -16                    # same magnitude as dW, so fp32 rounding of the sums stays relative
    base = torch.full((512, 64), b0, dtype=torch.float32, device=DEV)
    out2 = hip_loss(stage, case, "f32", dW=base.clone(), accumulate_dw=True)
    assert max_rel_err(out2["dW"].cpu().numpy(), b0 + ref["dW"]) <= TOL_F32


@pytest.mark.parametrize("n_tok,H,V", [
    (300, 128, 1000),        # ragged token tile, vocabulary not a multiple of the granule
    (256, 64, 256),          # exactly one tile
    (700, 256, 5000),        # several tiles each way
    (1, 64, 130),
])
def test_bf16_path_small_shapes(stage, n_tok, H, V):
    case = make_loss_case(100 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    check(out, ref, n_tok, TOL_BF16, case, all_zero=n_tok == 1)


def test_bf16_grad_scale_and_eps(stage):
    case = make_loss_case(7, 200, 128, 2000, "bf16", noise=0.3, w_std=0.1)
    ref = oracle_loss(**case, eps_lo=0.1, eps_hi=0.28, grad_scale=3.0)
    out = hip_loss(stage, case, "bf16", eps_lo=0.1, eps_hi=0.28, grad_scale=3.0)
    check(out, ref, 200, TOL_BF16, case)
    assert ((ref["r"] > 1.28) | (ref["r"] < 0.9)).sum() > 10


def test_bf16_peaked_softmax_and_unlikely_targets(stage):
    # logits with a spread of ~ +-20: half the targets are the arg-max (p close to 1, the one-hot
    # term nearly cancels), the rest are random (log(p_max / p_target) up to ~ 40, inside the bound of 70)
    import synth_inputs as si
    from oracle import grpo as ogrpo
    n_tok, H, V = 400, 128, 2000
    case = make_loss_case(31, n_tok, H, V, "bf16", noise=0.1, w_std=0.5)
    Z = case["hidden"].astype(np.float64) @ case["W"].astype(np.float64).T
    ids = case["ids"].copy()
    ids[::2] = Z[::2].argmax(axis=1)
    case["ids"] = ids.astype(np.int32)
    logp = ogrpo.token_logp(case["hidden"], case["W"], case["ids"])
    case["old_logp"] = (logp + np.random.default_rng(5).standard_normal(n_tok) * 0.1).astype(np.float32)
    gap = Z.max(axis=1) - Z[np.arange(n_tok), ids]
    assert gap.max() > 20 and gap.max() < 65 and (np.exp(logp[::2]) > 0.5).sum() > 50
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    check(out, ref, n_tok, TOL_BF16, case)


def test_bf16_multiple_chunks_and_accumulate(stage):
    import paper_2603_06619_amd as nat
    n_tok, H, V = 600, 128, 3000
    case = make_loss_case(8, n_tok, H, V, "bf16", noise=0.1, w_std=0.1)
    ref = oracle_loss(**case)
    ws_min = nat.loss_workspace_min_bytes(n_tok, H, V, nat.DTYPE_BF16)       # 256-token chunks -> 3 chunks
    out = hip_loss(stage, case, "bf16", ws_bytes=ws_min)
    check(out, ref, n_tok, TOL_BF16, case)
    b0 = float(np.abs(ref["dW"]).max())
    base = torch.full((V, H), b0, dtype=torch.float32, device=DEV)
    out2 = hip_loss(stage, case, "bf16", dW=base.clone(), accumulate_dw=True, ws_bytes=ws_min)
    assert max_rel_err(out2["dW"].cpu().numpy() - np.float32(b0), ref["dW"]) <= TOL_BF16


def test_bf16_deterministic_bitwise(stage):
    case = make_loss_case(9, 500, 128, 3000, "bf16", noise=0.1, w_std=0.1)
    a = hip_loss(stage, case, "bf16")
    a = {k: v.clone() for k, v in a.items()}
    b = hip_loss(stage, case, "bf16")
    for k in ("loss", "logp", "dH", "dW"):
        assert torch.equal(a[k], b[k]), k


def test_zero_kept_tokens(stage):
    import paper_2603_06619_amd as nat
    for tdt in (torch.bfloat16, torch.float32):
        W = torch.zeros((512, 64), dtype=tdt, device=DEV)
        dW = torch.full((512, 64), 7.0, dtype=torch.float32, device=DEV)
        loss = torch.full((1,), 3.0, dtype=torch.float32, device=DEV)
        nat.nat_loss_fwd_bwd(None, W, None, None, None, None, None, 0, 0.2, 0.2, 1.0, loss, None, None, dW, False, None)
        torch.cuda.synchronize()
        assert loss.item() == 0.0 and not dW.any()
        dW.fill_(7.0)
        nat.nat_loss_fwd_bwd(None, W, None, None, None, None, None, 0, 0.2, 0.2, 1.0, loss, None, None, dW, True, None)
        torch.cuda.synchronize()
        assert (dW == 7.0).all()


def test_bf16_qwen3_0p6b_head_reduced_batch(stage):
    # full head shape H=1024, V=151936; reduced batch (a few hundred kept tokens)
    case = make_loss_case(21, 300, 1024, 151936, "bf16")
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    errs = check(out, ref, 300, TOL_BF16, case, label="qwen3-0.6B head")
    print("qwen3-0.6B head reduced batch: rel err logp/dH/dW =", errs)


def test_bf16_qwen3_8b_head_reduced_batch(stage):
    # full head shape H=4096, V=151936; reduced batch
    case = make_loss_case(22, 130, 4096, 151936, "bf16")
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    errs = check(out, ref, 130, TOL_BF16, case, label="qwen3-8B head")
    print("qwen3-8B head reduced batch: rel err logp/dH/dW =", errs)


@pytest.mark.parametrize("H,V,label", [(5120, 151936, "wide head"), (3584, 152064, "Qwen2.5-Math-7B head")])
def test_bf16_other_full_head_shapes_reduced_batch(stage, H, V, label):
    # the remaining head shapes of the workloads: hidden sizes that are 20 and 14 tiles of 256 wide
    case = make_loss_case(23 + H, 150, H, V, "bf16")
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    errs = check(out, ref, 150, TOL_BF16, case, label=label)
    print(label, "reduced batch: rel err logp/dH/dW =", errs)


def test_bf16_hidden_size_not_a_multiple_of_the_tile(stage):
    # H = 320 (a multiple of 64 but not of 256): the last hidden tile is ragged in dH and dW
    case = make_loss_case(77, 300, 320, 1500, "bf16", noise=0.1, w_std=0.1)
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    check(out, ref, 300, TOL_BF16, case)


@pytest.mark.parametrize("n_tok", [31, 128, 129, 384, 385, 640])
def test_bf16_last_token_tile_half_full(stage, n_tok):
    # one token tile, half full or full, of a W that stays in the caches computes its first 64 or 128 columns of 256; tiles of several
    # columns are equal ones, 192 and 224 wide (logits, and dH whole and in ranges)
    for H, V in ((192, 1000), (64, 9000)):
        case = make_loss_case(500 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
        ref = oracle_loss(**case)
        check(hip_loss(stage, case, "bf16"), ref, n_tok, TOL_BF16, case)


@pytest.mark.parametrize("n_tok", [1, 64, 65, 320, 321])
def test_bf16_last_token_tile_a_quarter_full(stage, n_tok):
    # one token tile of at most 64 or 128 tokens, and two equal ones 160 and 192 wide; log-probs alone and with the loss are equal
    for H, V in ((192, 1000), (64, 9000)):
        case = make_loss_case(530 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
        out = hip_loss(stage, case, "bf16")
        check(out, oracle_loss(**case), n_tok, TOL_BF16, case)
        fwd = stage.logp(to_dev(case["hidden"], torch.bfloat16), to_dev(case["W"], torch.bfloat16), to_dev(case["ids"]), n_tok)
        assert torch.equal(fwd["logp"][:n_tok], out["logp"][:n_tok])


@pytest.mark.parametrize("n_tok", [1, 33, 65, 289, 353])
def test_bf16_workspace_contents_do_not_matter(stage, n_tok):
    # the contractions walk k-slices two at a time: with an odd number of 32-token slices dW reads one more than holds
    # tokens.  A workspace full of NaN bits gives the bits that a cleared one gives
    H, V = 192, 700
    case = make_loss_case(900 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    outs = []
    for byte in (0, 255):
        hip_loss(stage, case, "bf16")
        stage._ws["loss"].fill_(byte)
        outs.append(hip_loss(stage, case, "bf16"))
    for k in ("loss", "logp", "dH", "dW"):
        assert torch.equal(outs[0][k], outs[1][k]), k
    check(outs[1], oracle_loss(**case), n_tok, TOL_BF16, case)


@pytest.mark.parametrize("n_tok,H,V", [(200, 64, 65700), (500, 192, 65700), (7200, 64, 3000), (6200, 320, 3000)])
def test_bf16_workgroups_walk_several_tiles(stage, n_tok, H, V):
    # more tiles than compute units: a workgroup's load ring runs on from one tile into the next.  257 vocabulary tiles and
    # one or two token tiles with W read as it is, and 12 by 29 or 25 with W repacked; H = 64 has two k-slices per tile, so the
    # loads run two tiles ahead.  dW: 257 tiles of 8 and 16 slices
    case = make_loss_case(700 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    ref = oracle_loss(**case)
    check(hip_loss(stage, case, "bf16"), ref, n_tok, TOL_BF16, case)


@pytest.mark.parametrize("n_tok", [513, 769, 1025, 1124])
def test_bf16_nearly_empty_last_token_tile_of_several(stage, n_tok):
    # H = 64: three to five equal columns, and (1124) five of 256, whose short last tile the workgroups walk as a whole one;
    # entropies too, and the log-probs of the tokens in front of it have the bits that they have without it
    H, V = 64, 40000
    case = make_loss_case(560 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    ref = oracle_loss(**case)
    check(hip_loss(stage, case, "bf16"), ref, n_tok, TOL_BF16, case)
    hidden, W, ids = to_dev(case["hidden"], torch.bfloat16), to_dev(case["W"], torch.bfloat16), to_dev(case["ids"])
    whole = stage.logp(hidden, W, ids, n_tok, want_entropy=True)
    full = n_tok // 256 * 256
    front = stage.logp(hidden[:full], W, ids[:full], full, want_entropy=True)
    for k in ("logp", "entropy"):
        assert torch.equal(whole[k][:full], front[k][:full]), k


@pytest.mark.parametrize("H,V", [(64, 66000), (128, 700), (448, 66000)])
def test_bf16_tile_columns_of_every_width(stage, H, V):
    # up to six equal tile columns of 64, 128, 160, 192 or 224 tokens, four or six slices in flight, or columns of 256, with 2, 4 and 14 slices per tile
    # and walks of one or two: log-probs and entropies of the first n tokens have the bits that they have among 1800 (columns of 256)
    case = make_loss_case(800 + H, 1800, H, V, "bf16", noise=0.15, w_std=0.1)
    hidden, W, ids = to_dev(case["hidden"], torch.bfloat16), to_dev(case["W"], torch.bfloat16), to_dev(case["ids"])
    all_of_it = stage.logp(hidden, W, ids, 1800, want_entropy=True)
    for n in (1, 64, 65, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257, 320, 321, 384, 385, 449, 513, 577, 641, 672, 769, 896, 897, 1025, 1088,
              1089, 1281, 1344, 1537, 1568):
        for stored in stage._ws.values():
            stored.fill_(255)
        some = stage.logp(hidden[:n], W, ids[:n], n, want_entropy=True)
        for k in ("logp", "entropy"):
            assert torch.equal(some[k][:n], all_of_it[k][:n]), (n, k)


@pytest.mark.parametrize("n_tok", [40, 100, 161, 260, 321, 448, 513, 640, 800, 1025, 1300])
@pytest.mark.parametrize("H,V", [(64, 4000), (320, 1500)])
def test_bf16_gradients_of_every_column_width(stage, n_tok, H, V):
    # dH and dW where the token columns are 64, 128 (dH alone; the logits of so small a W are not), 192, 160, 192, 224, 192, 224, 224, 224 and 224 wide,
    # one to six of them
    case = make_loss_case(840 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    hip_loss(stage, case, "bf16")
    stage._ws["loss"].fill_(255)
    check(hip_loss(stage, case, "bf16"), oracle_loss(**case), n_tok, TOL_BF16, case)


@pytest.mark.parametrize("n_tok,H,V", [
    (1124, 192, 3000),       # five columns, 100 tokens in the last: its first 128 columns
    (1100, 320, 17000),      # more tiles than compute units
    (1800, 448, 3000),       # eight columns, 8 tokens in the last: its first 64
    (1580, 4160, 1000),      # seven columns, 44 in the last, 130 slices per tile
    (600, 4160, 22100),      # three columns that are no equal ones: more tiles than compute units and more than 128 slices
])
def test_bf16_short_last_token_tile_beside_whole_ones(stage, n_tok, H, V):
    # a last token tile with at most 128 or 64 tokens has workgroups of its own that compute only its first 128 or 64 columns.  Loss and
    # gradients of all tokens against the oracle, and the entropies of those in the last tile
    case = make_loss_case(870 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1 if H < 4096 else 0.02)
    hip_loss(stage, case, "bf16")
    stage._ws["loss"].fill_(255)
    out = hip_loss(stage, case, "bf16", want_entropy=True)
    ref = oracle_loss(**case)
    check(out, ref, n_tok, TOL_BF16, case)
    last = slice((n_tok - 1) // 256 * 256, n_tok)
    assert max_rel_err(out["dH"][last].float().cpu().numpy(), ref["dH"][last]) <= TOL_BF16
    from oracle import grpo as ogrpo
    ent = ogrpo.forward_logp(case["hidden"][last], case["W"], case["ids"][last])["entropy"]
    assert max_rel_err(out["entropy"][last].cpu().numpy(), ent) <= 1e-4


def accumulated_and_plain(stage, n_tok, H, V):
    case = make_loss_case(600 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.1)
    plain = hip_loss(stage, case, "bf16")["dW"]
    big = torch.randn((V + 1, H), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV) * plain.abs().mean()
    old = big.clone()
    acc = hip_loss(stage, case, "bf16", dW=big[:V], accumulate_dw=True)["dW"]
    assert torch.equal(acc, old[:V] + plain)
    assert torch.equal(big[V], old[V])
    return case, plain


@pytest.mark.parametrize("V", [1025, 17153])
@pytest.mark.parametrize("n_tok", [40, 2048, 2049])
def test_bf16_accumulating_equals_old_plus_overwritten(stage, n_tok, V):
    # a chunk is added to dW by reading, adding and storing, in the contraction or, for tiles whose token axis is cut, in the kernel that
    # sums their ranges.  V = 17153: 136 tiles, more than half a round of compute units, so none is cut; V = 1025: 10 tiles, all cut
    # from 2048 tokens on.  One addition of the same sum per element either way, so accumulating equals old + the overwritten result
    # bit for bit.  Columns and rows past the end of the last tiles (H = 320, one row in the last tile) keep what they held
    accumulated_and_plain(stage, n_tok, 320, V)


@pytest.mark.parametrize("n_tok", [200, 2100])
def test_bf16_accumulating_where_workgroups_walk(stage, n_tok):
    # 257 dW tiles, so that a workgroup's old values and stores come between the next tile's loads: 8 slices each, and 66, where the
    # 257th is cut into two ranges and a walk goes from a whole tile to a range
    case, plain = accumulated_and_plain(stage, n_tok, 64, 65700)
    if n_tok == 200:
        assert max_rel_err(plain.cpu().numpy(), oracle_loss(**case)["dW"]) <= TOL_BF16


@pytest.mark.parametrize("n_tok", [8192, 8193])
def test_bf16_dw_where_walks_end(stage, n_tok):
    # 258 dW tiles of 256 k-slices are walked, of 258 not.  Against the sum of calls over half the tokens, whose products are the same
    # and whose fp32 sums run in another order: 512 additions of relative 2^-24 each, with random signs 1.4e-6
    H, V = 320, 33000
    case, plain = accumulated_and_plain(stage, n_tok, H, V)
    dW = torch.zeros((V, H), device=DEV)
    for half in (slice(0, 4096), slice(4096, n_tok)):
        part = {k: (v[half] if k in ("hidden", "ids", "old_logp", "kept_seq", "kept_w") else v) for k, v in case.items()}
        hip_loss(stage, part, "bf16", dW=dW, accumulate_dw=True)
    assert float((plain - dW).norm() / dW.norm()) <= 1e-5


@pytest.mark.parametrize("V", [61680, 61681])
def test_bf16_dw_at_the_line_where_it_passes_the_caches(stage, V):
    # 1088 x 61680 x 4 bytes are the last below 256 MiB; whole tiles and, in both directions, cut ones
    case, plain = accumulated_and_plain(stage, 40, 1088, V)
    assert max_rel_err(plain.cpu().numpy(), oracle_loss(**case)["dW"]) <= TOL_BF16


@pytest.mark.parametrize("H,V,n", [(64, 7, 6144), (320, 700, 6144), (192, 1025, 6144), (256, 700, 7168)])
def test_bf16_w_repacked_and_read_as_it_is_agree(stage, H, V, n):
    # up to n tokens the contractions read W in place, beyond that a repacked copy: the same products in the same
    # order, so the log-probs of the common tokens are equal bit for bit, and each side meets the path's tolerance
    case = make_loss_case(77, n + 1, H, V, "bf16", noise=0.15, w_std=0.1)
    short = {k: (v[:n] if k in ("hidden", "ids", "old_logp", "kept_seq", "kept_w") else v) for k, v in case.items()}
    packed, direct = hip_loss(stage, case, "bf16"), hip_loss(stage, short, "bf16")
    assert torch.equal(packed["logp"][:n], direct["logp"][:n])
    check(direct, oracle_loss(**short), n, TOL_BF16, short)
    check(packed, oracle_loss(**case), n + 1, TOL_BF16, case)
    fwd = stage.logp(to_dev(case["hidden"], torch.bfloat16), to_dev(case["W"], torch.bfloat16), to_dev(case["ids"]), n + 1)
    assert torch.equal(fwd["logp"][:n + 1], packed["logp"][:n + 1])


@pytest.mark.parametrize("H,V,n", [(64, 700, 8192), (192, 1025, 8192), (256, 300, 24576)])
def test_bf16_forward_pass_w_repacked_and_read_as_it_is_agree(stage, H, V, n):
    # the same for the forward pass alone: the common tokens' log-probs and entropies, bit for bit
    case = make_loss_case(78, n + 1, H, V, "bf16", noise=0.15, w_std=0.1)
    hidden, W, ids = to_dev(case["hidden"], torch.bfloat16), to_dev(case["W"], torch.bfloat16), to_dev(case["ids"])
    packed = {k: v.clone() for k, v in stage.logp(hidden, W, ids, n + 1, want_entropy=True).items() if v is not None}
    direct = stage.logp(hidden[:n], W, ids[:n], n, want_entropy=True)
    assert torch.equal(packed["logp"][:n], direct["logp"][:n])
    assert torch.equal(packed["entropy"][:n], direct["entropy"][:n])


@pytest.mark.parametrize("n_tok,H,V,label", [
    (4700, 3584, 2100, "dH: a full round of tiles and ten more in two vocabulary ranges"),
    (100, 128, 40000, "dH: one tile in 37 vocabulary ranges"),
    (257, 320, 9000, "dH: four tiles, two of them with one valid row, in nine ranges"),
])
def test_bf16_dh_leftover_tiles_cut_into_vocabulary_ranges(stage, n_tok, H, V, label):
    case = make_loss_case(300 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.02)
    ref = oracle_loss(**case)
    check(hip_loss(stage, case, "bf16"), ref, n_tok, TOL_BF16, case, label=label)


@pytest.mark.parametrize("n_tok,H,V", [(150, 64, 30000), (190, 320, 9000), (300, 1024, 9000), (420, 256, 9000), (530, 576, 5000), (1070, 128, 4200),
                                       (330, 4160, 3000)])
def test_bf16_dh_of_narrow_columns_in_ranges(stage, n_tok, H, V):
    # dH of one to five equal tile columns of 160 to 224 tokens, its vocabulary cut into ranges: numbers of tiles and of units that
    # do and do not divide by the 8 XCDs (1, 2, 8, 2, 9, 5, 34 tiles).  Two runs agree bit for bit
    case = make_loss_case(320 + n_tok, n_tok, H, V, "bf16", noise=0.15, w_std=0.02)
    out = hip_loss(stage, case, "bf16")
    check(out, oracle_loss(**case), n_tok, TOL_BF16, case)
    first = out["dH"].clone()
    stage._ws["loss"].fill_(255)
    assert torch.equal(first, hip_loss(stage, case, "bf16")["dH"])


def test_bf16_dw_leftover_tiles_cut_into_token_ranges(stage):
    # 8 dW tiles on 256 compute units: all of them are "left over" after the last full round, so the library
    # cuts their token axis (8173 tokens = 256 k-slices) into 8 ranges and adds the partial tiles in range
    # order; checked against the oracle element by element, with and without accumulation, and bit for bit
    # between two runs
    n_tok, H, V = 8192 - 19, 256, 2048
    case = make_loss_case(55, n_tok, H, V, "bf16", noise=0.1, w_std=0.1)
    ref = oracle_loss(**case)
    out = hip_loss(stage, case, "bf16")
    check(out, ref, n_tok, TOL_BF16, case, label="dW tiles in 8 token ranges")
    first = out["dW"].clone()
    b0 = float(np.abs(ref["dW"]).max())
    base = torch.full((V, H), b0, dtype=torch.float32, device=DEV)
    out2 = hip_loss(stage, case, "bf16", dW=base.clone(), accumulate_dw=True)
    assert max_rel_err(out2["dW"].cpu().numpy() - np.float32(b0), ref["dW"]) <= TOL_BF16
    again = hip_loss(stage, case, "bf16")
    assert torch.equal(first, again["dW"])


def test_bf16_full_vocabulary_mid_size_every_element_of_dw(stage):
    # the whole vocabulary (V = 151936, H = 1024) with enough tokens for 9 token tiles, and a workspace
    # that forces 3 chunks: dW (and everything else) against the oracle element by element
    import paper_2603_06619_amd as nat
    n_tok, H, V = 2304 - 37, 1024, 151936                  # ragged last token tile
    case = make_loss_case(301, n_tok, H, V, "bf16")
    ref = oracle_loss(**case)
    ws = nat.loss_workspace_bytes(768, H, V, nat.DTYPE_BF16) + 64 * 1024     # room for 768-token chunks, not 1024
    assert ws < nat.loss_workspace_bytes(1024, H, V, nat.DTYPE_BF16)
    out = hip_loss(stage, case, "bf16", ws_bytes=ws)
    check(out, ref, n_tok, TOL_BF16, case, label="full vocabulary, H = 1024, %d tokens in 3 chunks" % n_tok)
    # one chunk gives the same log-probs bit for bit and dW within rounding of the chunked sum (with one chunk
    # the 72 dW tiles left over after 9 full rounds are cut into two token ranges)
    one = hip_loss(stage, case, "bf16")
    assert torch.equal(one["logp"][:n_tok], out["logp"][:n_tok])
    check(one, ref, n_tok, TOL_BF16, case, label="same, one chunk")
