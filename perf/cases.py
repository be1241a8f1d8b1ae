"""The timed cases of the partial-token GRPO loss stage: what a training program has it do.

Four kinds of call, each through the package's public entry points:

  step    one optimiser step's worth of the stage: advantages -> selection -> compaction with the
          gather of the kept rows -> loss and gradients (`LossStage`, as `bench.py` drives it);
  loss    loss and gradients on kept tokens that are already gathered, in one or more micro-batches
          whose dW accumulates (the first call overwrites, the later ones add);
  logp    the forward pass alone (behaviour and reference log-probs, entropies);
  select  selection and compaction alone, on buffers that the program keeps (a loop that selects for
          a body it runs elsewhere), optionally with the truncated batch for that body.

Heads, group sizes, length laws and selection schemes are those of `synth_inputs.WORKLOADS` and of
`bench.py`; the small heads are those of the tests.
"""
import math

import numpy as np
import torch

import paper_2603_06619_amd as nat
from paper_2603_06619_amd.stage import LossStage

DEV = "cuda:0"
W_STD = 0.02            # head weights ~ N(0, 0.02), hidden states ~ N(0, 1)
LOGP_NOISE = 0.05       # behaviour log-probs = current log-probs + N(0, 0.05)
SCHEMES = {"full": nat.FULL, "urs": nat.URS, "rpc": nat.RPC, "det": nat.DET, "mixed": nat.URS}

# (H, V) of the full-size heads: 0.6B, 8B, wide-head stress, Qwen2.5-Math-7B
HEADS = [(1024, 151936), (4096, 151936), (5120, 151936), (3584, 152064)]


def listed():
    return [
        # the tiny fp32 workload as a whole: nothing but latency and launches
        dict(name="tiny_fp32_step", kind="step", dtype="f32", H=64, V=512, P=2, G=4, law="uniform", lo=16, hi=64,
             scheme="urs", p=0.5, C=1, drop=False),
        # an fp32 gradient check on a reduced head: ragged token count
        dict(name="fp32_loss_reduced_head", kind="loss", dtype="f32", H=256, V=4096, tokens=601, micro=1, kl="none",
             entropy=False),
        # the 0.6B head's whole step (short contraction: K = 1024), URS 1/2
        dict(name="step_0p6b_urs", kind="step", dtype="bf16", H=1024, V=151936, P=8, G=8, law="uniform", lo=256,
             hi=2048, scheme="urs", p=0.5, C=1, drop=False),
        # log-probs of one short rollout at the 0.6B head: the smallest forward call, one ragged token tile
        dict(name="logp_0p6b_one_rollout", kind="logp", dtype="bf16", H=1024, V=151936, tokens=301, entropy=False),
        # gradient accumulation at the 8B head: two ragged micro-batches of about one kept rollout each
        dict(name="loss_8b_micro_batches", kind="loss", dtype="bf16", H=4096, V=151936, tokens=1237, micro=2,
             kl="none", entropy=False),
        # one prompt's group of rollouts at the Qwen2.5-Math-7B head with the KL term and the entropy
        dict(name="loss_7b_kl_entropy", kind="loss", dtype="bf16", H=3584, V=152064, tokens=5003, micro=1,
             kl="nonneg", entropy=True),
        # behaviour log-probs and entropies of a few rollouts at the 8B head
        dict(name="logp_8b_entropy", kind="logp", dtype="bf16", H=4096, V=151936, tokens=12289, entropy=True),
        # wide head, heavy-tailed lengths, URS and deterministic truncation mixed in one batch
        dict(name="step_wide_mixed", kind="step", dtype="bf16", H=5120, V=151936, P=8, G=8, law="pareto", lo=128,
             hi=32768, scheme="mixed", p=0.5, C=1, drop=False),
        # the headline workload, whole: 8B head, RPC, 16 prompts x 8 rollouts
        dict(name="step_8b_rpc", kind="step", dtype="bf16", H=4096, V=151936, P=16, G=8, law="lognormal", lo=2048,
             hi=8192, scheme="rpc", p=0.5, C=1, drop=False),
        # selection alone for a long chain-of-thought batch: 128 rollouts, 1.3 million tokens
        dict(name="select_long_cot_rpc", kind="select", B=128, law="uniform", lo=4096, hi=16384, scheme="rpc", p=0.5,
             C=100, pack=False),
        # a cut schedule with explicit survival probabilities, and the truncated batch for the body
        dict(name="select_schedule_pack", kind="select", B=128, law="lognormal", lo=2048, hi=8192, scheme="schedule",
             p=0.5, C=1, pack=True),
        # selection on an inflated batch with per-token probabilities: 4096 rollouts, 2^26 tokens
        dict(name="select_poisson_large", kind="select", B=4096, law="uniform", lo=1, hi=32767, scheme="poisson",
             p=0.5, C=1, pack=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step_f32", "loss_f32", "step", "loss", "loss", "logp", "select", "select"])
    if kind == "step_f32":
        lo = rng.randint(1, 32)
        return dict(kind="step", dtype="f32", H=4 * rng.randint(12, 64), V=_log_int(rng, 300, 4096), P=rng.randint(1, 4),
                    G=rng.randint(2, 8), law="uniform", lo=lo, hi=lo + rng.randint(0, 64),
                    scheme=rng.choice(["urs", "rpc", "full", "det"]), p=rng.choice([0.25, 0.5, 0.9]), C=1, drop=False)
    if kind == "loss_f32":
        return dict(kind="loss", dtype="f32", H=4 * rng.randint(12, 64), V=_log_int(rng, 300, 4096),
                    tokens=_log_int(rng, 16, 1024), micro=rng.randint(1, 2),
                    kl=rng.choice(["none", "log_ratio", "nonneg"]), entropy=rng.random() < 0.5)
    if kind == "step":
        H, V = rng.choice(HEADS)
        G = rng.choice([4, 8, 16])
        # tokens of the batch, over the logarithm; the largest stays below the headline workload
        mean_len = _log_int(rng, 128, 4096)
        P = max(1, min(32, _log_int(rng, 1500, 100000) // (G * mean_len)))
        law = rng.choice(["uniform", "lognormal", "pareto"])
        lo = {"uniform": max(1, mean_len // 4), "lognormal": mean_len, "pareto": max(1, mean_len // 3)}[law]
        hi = {"uniform": mean_len * 7 // 4, "lognormal": 4 * mean_len, "pareto": 16 * mean_len}[law]
        return dict(kind="step", dtype="bf16", H=H, V=V, P=P, G=G, law=law, lo=lo, hi=hi,
                    scheme=rng.choice(["urs", "rpc", "mixed", "det", "full"]), p=rng.choice([0.25, 0.5, 0.75]),
                    C=rng.choice([1, 100]), drop=P >= 4 and rng.random() < 0.3)
    if kind in ("loss", "logp"):
        if rng.random() < 0.25:                       # a head of some other model: any vocabulary size
            H, V = 64 * rng.randint(1, 48), _log_int(rng, 1000, 160000)
        else:
            H, V = rng.choice(HEADS)
        tokens = _log_int(rng, 32, 32768)
        if kind == "logp":
            return dict(kind="logp", dtype="bf16", H=H, V=V, tokens=tokens, entropy=rng.random() < 0.5)
        return dict(kind="loss", dtype="bf16", H=H, V=V, tokens=tokens, micro=rng.choice([1, 1, 2, 3]),
                    kl=rng.choice(["none", "none", "log_ratio", "nonneg"]), entropy=rng.random() < 0.3)
    scheme = rng.choice(["urs", "rpc", "det", "mixed", "schedule", "poisson"])
    hi = _log_int(rng, 16, 32767)
    lo = rng.randint(0, hi // 2)
    B = max(1, min(4096, _log_int(rng, 1000, 1 << 26) // hi))
    return dict(kind="select", B=B, law="uniform", lo=lo, hi=hi, scheme=scheme, p=rng.choice([0.1, 0.25, 0.5, 0.9]),
                C=rng.choice([1, 100]), pack=scheme in ("rpc", "det", "schedule") and rng.random() < 0.5)


# ------------------------------------------------------------------ inputs ----
def _lengths(case, n, rng):
    lo, hi = case["lo"], case["hi"]
    if case["law"] == "uniform":
        T = rng.integers(lo, hi + 1, size=n)
    elif case["law"] == "lognormal":                  # median lo, sigma 0.5, capped at hi
        T = np.clip(np.rint(np.exp(rng.normal(math.log(lo), 0.5, size=n))), 1, hi)
    else:                                             # Pareto, alpha 1.5, minimum lo, capped at hi
        T = np.clip(np.floor(lo * (1.0 - rng.random(size=n)) ** (-1.0 / 1.5)), 1, hi)
    return T.astype(np.int64)


def _layout(case):
    """Response lengths and packed offsets: they belong to the case, so that every seed gives the same shapes."""
    B = case["B"] if case["kind"] == "select" else case["P"] * case["G"]
    T = _lengths(case, B, np.random.default_rng([11, B]))
    return T, np.concatenate([[0], np.cumsum(T)]).astype(np.int64)


def _kept_share(case):
    s = case["scheme"]
    if s == "full":
        return 1.0
    if s == "urs":
        return case["p"]
    if s == "poisson":
        return 0.43                                   # mean of 0.9 (0.05 + 0.95 u^2) + 0.1
    if s == "schedule":
        return 2.0 / 3.0                              # half the mass spread over the positions, a third on the last
    return 0.5                                        # rpc (C = 1), det (1/2), mixed


_stage = None


def _the_stage():
    """One stage per program: it keeps the workspaces."""
    global _stage
    if _stage is None:
        _stage = LossStage(DEV)
    return _stage


def _head(case, gen):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    W = torch.empty((case["V"], case["H"]), device=DEV, dtype=dt)
    for v0 in range(0, case["V"], 16384):
        rows = min(16384, case["V"] - v0)
        W[v0:v0 + rows] = torch.randn((rows, case["H"]), generator=gen, device=DEV) * W_STD
    return W


def _hidden(n, case, gen):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    h = torch.empty((n, case["H"]), device=DEV, dtype=dt)
    for k0 in range(0, n, 65536):
        rows = min(65536, n - k0)
        h[k0:k0 + rows] = torch.randn((rows, case["H"]), generator=gen, device=DEV)
    return h


def _old_logp(hidden, W, ids, gen):
    """Behaviour log-probs: the current ones plus N(0, 0.05).  The current log-prob is z_y - log-sum-exp; for
    Gaussian weights the log-sum-exp is log V + |0.02 h|^2 / 2 to within the sampling error of V terms."""
    n = hidden.shape[0]
    out = torch.empty(n, device=DEV, dtype=torch.float32)
    for k0 in range(0, n, 32768):
        h = hidden[k0:k0 + 32768].float()
        z = (h * W[ids[k0:k0 + 32768].long()].float()).sum(1)
        out[k0:k0 + 32768] = z - (math.log(W.shape[0]) + 0.5 * W_STD ** 2 * h.square().sum(1))
    return out + LOGP_NOISE * torch.randn(n, generator=gen, device=DEV)


def _schemes(case, B):
    if case["scheme"] != "mixed":                     # mixed: even prompts URS, odd prompts deterministic truncation
        return None
    return np.where((np.arange(B) // case.get("G", 8)) % 2 == 0, nat.URS, nat.DET).astype(np.int32)


def _params(case, seed, spr):
    code = SCHEMES.get(case["scheme"], nat.FULL)
    return nat.SelectParams(code, p=case["p"], min_cut=case["C"], trunc_frac=0.5, seed=seed, step=3,
                            scheme_per_rollout=None if spr is None else torch.from_numpy(spr).to(DEV))


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng([seed, 1])
    s = dict(case=case, seed=seed)
    if case["kind"] == "select":
        B = case["B"]
        T, cu = _layout(case)
        spr, N = _schemes(case, B), int(cu[-1])
        i32 = lambda n: torch.zeros(max(int(n), 1), dtype=torch.int32, device=DEV)
        s.update(B=B, N=N, cu_host=cu, spr_host=spr, cu=torch.from_numpy(cu).to(DEV), params=_params(case, seed, spr),
                 ids=torch.randint(0, 151936, (max(N, 1),), generator=gen, device=DEV, dtype=torch.int32),
                 old_logp=-12.0 + torch.randn(max(N, 1), generator=gen, device=DEV),
                 cut_len=i32(B), mask=i32(nat.mask_words(N)), kept_idx=i32(N), kept_seq=i32(N), ids_k=i32(N),
                 kept_w=torch.zeros(max(N, 1), device=DEV), old_logp_k=torch.zeros(max(N, 1), device=DEV),
                 cu_kept=i32(B + 1), n_kept=i32(1), h_n_kept=torch.zeros(1, dtype=torch.int32).pin_memory(),
                 ws=torch.empty(nat.compact_workspace_bytes(N), dtype=torch.uint8, device=DEV))
        if case["scheme"] == "poisson":               # about 10 % of the tokens at exactly 1
            pi = 0.05 + 0.95 * torch.rand(max(N, 1), generator=gen, device=DEV, dtype=torch.float64).square()
            pi[torch.rand(max(N, 1), generator=gen, device=DEV) < 0.1] = 1.0
            s["pi"] = pi
        if case["scheme"] == "schedule":              # ones, and a point mass of T // 2 on the last position
            w = np.ones(max(N, 1), dtype=np.int32)
            w[cu[1:][T > 0] - 1] += (T[T > 0] // 2).astype(np.int32)
            s["weights"] = torch.from_numpy(w).to(DEV)
            s["pi"] = torch.zeros(max(N, 1), dtype=torch.float64, device=DEV)
        if case["pack"]:
            plen = np.random.default_rng([12, B]).integers(32, 513, B).astype(np.int32)
            rows = N + int(plen.sum())
            s.update(prompt_len=torch.from_numpy(plen).to(DEV), rows_cap=rows, cu_packed=i32(B + 1), cu_loss=i32(B + 1),
                     src_idx=i32(rows), position_ids=i32(rows), loss_row=i32(N), totals=i32(2),
                     h_totals=torch.zeros(2, dtype=torch.int32).pin_memory(),
                     input_ids=torch.randint(0, 151936, (rows,), generator=gen, device=DEV, dtype=torch.int32),
                     input_ids_packed=i32(rows))
        return s

    s["stage"] = _the_stage()
    s["W"] = _head(case, gen)
    if case["kind"] == "step":
        P, G = case["P"], case["G"]
        B = P * G
        T, cu = _layout(case)
        spr, N = _schemes(case, B), int(cu[-1])
        # binary rewards, half of each group right; with all-equal groups in a tenth to a quarter of the prompts
        R = rng.permuted(np.tile((np.arange(G) % 2).astype(np.float32), (P, 1)), axis=1)
        if case["drop"] or (case["scheme"] == "mixed" and P >= 4):
            n_eq = math.ceil((0.25 if case["drop"] else 0.1) * P)
            R[:n_eq] = R[:n_eq, :1]
        # the draw of one training step: the same tokens whatever the inputs, so that shapes stay
        s.update(B=B, N=N, cu_host=cu, spr_host=spr, R=R, rewards=torch.from_numpy(R.reshape(-1)).to(DEV),
                 cu=torch.from_numpy(cu).to(DEV), seed=2000, params=_params(case, 2000, spr))
        n_tok = N
    else:
        n_tok = case["tokens"] * case.get("micro", 1)
    s["hidden"] = _hidden(n_tok, case, gen)
    s["ids"] = torch.randint(0, case["V"], (n_tok,), generator=gen, device=DEV, dtype=torch.int32)
    if case["kind"] != "logp":
        s["old_logp"] = _old_logp(s["hidden"], s["W"], s["ids"], gen)
        s["dW"] = torch.zeros((case["V"], case["H"]), device=DEV)
    if case["kind"] == "loss":
        # kept tokens of eight rollouts: random-prefix weights 1 / (B T p) with p falling to 1 / T, advantages of
        # binary rewards; the reference policy is a little further off than the behaviour policy
        n_seq = 8
        seq = np.sort(rng.integers(0, n_seq, n_tok)).astype(np.int32)
        adv = np.where(rng.random(n_seq) < 0.5, 1.0, -1.0) * rng.uniform(0.4, 2.5, n_seq)
        s["adv"] = torch.from_numpy(adv.astype(np.float32)).to(DEV)
        s["kept_seq"] = torch.from_numpy(seq).to(DEV)
        s["kept_w"] = torch.from_numpy((1.0 / (128 * 2048 * rng.uniform(0.05, 1.0, n_tok))).astype(np.float32)).to(DEV)
        if case["kl"] != "none":
            s["ref_logp"] = s["old_logp"] + 2 * LOGP_NOISE * torch.randn(n_tok, generator=gen, device=DEV)
    return s


# -------------------------------------------------------------------- run ----
def _run_select(s):
    case, B, N = s["case"], s["B"], s["N"]
    compact = (s["kept_idx"], s["kept_seq"], s["kept_w"], s["cu_kept"], s["n_kept"], s["h_n_kept"], s["ws"])
    gather = dict(ids=s["ids"], ids_k=s["ids_k"], old_logp=s["old_logp"], old_logp_k=s["old_logp_k"])
    if case["scheme"] == "poisson":
        nat.nat_select_poisson(s["params"], s["pi"], s["cu"], B, N, s["mask"])
        nat.nat_compact_pi(B, s["mask"], s["pi"], s["cu"], B, N, *compact, **gather)
    elif case["scheme"] == "schedule":
        nat.nat_select_schedule(s["params"], s["weights"], s["cu"], B, N, s["cut_len"], s["mask"], s["pi"])
        nat.nat_compact_pi(B, s["mask"], s["pi"], s["cu"], B, N, *compact, **gather)
    else:
        nat.nat_select(s["params"], s["cu"], B, N, s["cut_len"], s["mask"])
        nat.nat_compact(s["params"], B, s["mask"], s["cu"], B, N, *compact, **gather)
    keys = ["mask", "kept_idx", "kept_seq", "kept_w", "cu_kept", "n_kept", "ids_k", "old_logp_k"]
    if case["scheme"] != "poisson":
        keys.append("cut_len")
    if case["scheme"] == "schedule":
        keys.append("pi")
    if case["pack"]:
        nat.nat_prefix_pack(s["prompt_len"], s["cu"], s["cut_len"], B, 1, s["rows_cap"], N, s["cu_packed"],
                            s["cu_loss"], s["src_idx"], s["position_ids"], s["loss_row"], s["totals"], s["h_totals"],
                            s["input_ids"], s["input_ids_packed"])
        keys += ["cu_packed", "cu_loss", "src_idx", "position_ids", "loss_row", "totals", "input_ids_packed"]
    return {k: s[k] for k in keys}


def run(state):
    s, case = state, state["case"]
    if case["kind"] == "select":
        return _run_select(s)
    stage = s["stage"]
    if case["kind"] == "logp":
        out = stage.logp(s["hidden"], s["W"], s["ids"], case["tokens"], want_entropy=case["entropy"])
        return dict(logp=out["logp"], entropy=out["entropy"])
    if case["kind"] == "step":
        adv = stage.advantage(s["rewards"], case["P"], case["G"])
        s["params"].drop_zero_adv = adv if case["drop"] else None
        sc = stage.select_compact(s["params"], s["cu"], s["B"], s["N"], hidden=s["hidden"], ids=s["ids"],
                                  old_logp=s["old_logp"])
        nk = sc["n_kept"]
        out = stage.loss(sc["hidden_k"], s["W"], sc["ids_k"], sc["old_logp_k"], adv, sc["kept_seq"], sc["kept_w"], nk,
                         dW=s["dW"])
        return dict(adv=adv, kept_idx=sc["kept_idx"][:nk], kept_w=sc["kept_w"][:nk], loss=out["loss"],
                    logp=out["logp"][:nk], dH=out["dH"][:nk], dW=out["dW"])
    parts, n = [], case["tokens"]
    for m in range(case["micro"]):
        k = slice(m * n, (m + 1) * n)
        kl = {}
        if case["kl"] != "none":
            kl = dict(ref_logp_k=s["ref_logp"][k], beta_kl=0.04, want_kl=True,
                      kl_kind=nat.KL_NONNEG if case["kl"] == "nonneg" else nat.KL_LOG_RATIO)
        out = stage.loss(s["hidden"][k], s["W"], s["ids"][k], s["old_logp"][k], s["adv"], s["kept_seq"][k],
                         s["kept_w"][k], n, dW=s["dW"], accumulate_dw=m > 0, want_entropy=case["entropy"], **kl)
        parts.append({q: out.get(q) for q in ("loss", "logp", "dH", "kl", "entropy")})
    return dict(parts=parts, dW=s["dW"])


# ------------------------------------------------------------------- work ----
def work(case):
    if case["kind"] == "select":
        N = float(_layout(case)[1][-1])
        nk = N * _kept_share(case)
        b = N / 8 + 28.0 * nk                         # mask out; index, rollout, weight, two gathered pairs
        if case["scheme"] == "poisson":
            b += 8.0 * N                              # probabilities in
        if case["scheme"] == "schedule":
            b += 12.0 * N                             # weights in, probabilities out
        if case["pack"]:
            b += 16.0 * (nk + 272.0 * case["B"]) + 4.0 * nk
        return {"bytes": b, "flops": 0}
    el = 2 if case["dtype"] == "bf16" else 4
    H, V = case["H"], case["V"]
    if case["kind"] == "logp":
        n = case["tokens"]
        return {"bytes": el * H * (n + V) + 8.0 * n, "flops": 2.0 * V * H * n}
    extra = 0.0
    if case["kind"] == "step":
        N = float(_layout(case)[1][-1])
        n = N * _kept_share(case)
        extra = N / 8 + 28.0 * n
        if case["scheme"] == "rpc" and case["C"] > 1:
            n += 0.5 * case["C"] * case["P"] * case["G"]
        if case["drop"]:
            n *= 0.75
    else:
        n = case["tokens"] * case["micro"]
    # hidden rows in, head in, dH out, dW (fp32) out
    return {"bytes": extra + el * H * (2.0 * n + V) + 4.0 * V * H + 24.0 * n, "flops": 6.0 * V * H * n}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    if case["kind"] == "logp":                        # single-precision sums: 9e-8 off the 64-bit values
        return {"rel": 4e-7, "max": 2e-5}
    if case["dtype"] == "f32":                        # single precision: dH 1.3e-6, loss 2e-6 where its terms cancel;
        return {"rel": 3e-5 if case.get("kl", "none") != "none" else 1e-5, "max": 1e-3}   # the KL term (small) 7e-6
    # the soft-max numerators and the scaled hidden rows are rounded to bf16 once each (2.3e-3 to 2.5e-3)
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------ exact ----
def _philox(c0, c1, c2, c3, key0, key1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words (Salmon et al., SC'11)."""
    m32 = 0xFFFFFFFF
    for r in range(10):
        k0, k1 = (key0 + r * 0x9E3779B9) & m32, (key1 + r * 0xBB67AE85) & m32
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57     # low 64 bits; the shifts below are masked
        c0, c1, c2, c3 = ((p1 >> 32) & m32) ^ c1 ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c3 ^ k1, p0 & m32
    return c0, c1, c2, c3


def _exact_selection(s, adv=None):
    """(kept positions, rollouts, weights in 64 bits, probabilities or None)."""
    case, B, N = s["case"], s["B"], s["N"]
    key0, key1 = s["seed"] & 0xFFFFFFFF, s["seed"] >> 32
    T = torch.from_numpy(np.diff(s["cu_host"])).to(DEV)
    seq = torch.repeat_interleave(torch.arange(B, device=DEV), T)
    t0 = torch.arange(N, device=DEV) - s["cu"][seq]
    Tn = T[seq]
    dbl = lambda x: x.to(torch.float64)
    zero = lambda like: torch.zeros_like(like)
    code = SCHEMES.get(case["scheme"], nat.FULL)
    scheme = torch.full((B,), code, device=DEV) if s["spr_host"] is None else torch.from_numpy(s["spr_host"]).to(DEV).long()
    pi = None
    if case["scheme"] in ("urs", "mixed", "poisson"):
        words = torch.stack(_philox(t0 >> 2, seq, zero(t0), torch.full_like(t0, 3), key0, key1), 1)
        word = words.gather(1, (t0 & 3)[:, None])[:, 0]
    ids = torch.arange(B, device=DEV)
    if case["scheme"] == "poisson":
        pi = s["pi"][:N]
        keep = word < torch.floor(pi * 4294967296.0).long()
        w = 1.0 / (dbl(B * Tn) * pi)
    elif case["scheme"] == "schedule":
        x, y, _, _ = _philox(zero(ids), ids, torch.full_like(ids, 2), torch.full_like(ids, 3), key0, key1)
        a = s["weights"][:N].cpu().numpy().astype(np.int64)
        cut, surv = np.zeros(B, np.int64), np.zeros(N, np.float64)
        for i in range(B):
            lo, hi = int(s["cu_host"][i]), int(s["cu_host"][i + 1])
            if hi == lo:
                continue
            run_sum = np.cumsum(a[lo:hi])
            A = int(run_sum[-1])
            r = (((int(x[i]) << 32) | int(y[i])) * A) >> 64
            cut[i] = int(np.searchsorted(run_sum, r, side="right")) + 1
            surv[lo:hi] = (A - run_sum + a[lo:hi]) / A
        pi = torch.from_numpy(surv).to(DEV)
        keep = t0 < torch.from_numpy(cut).to(DEV)[seq]
        w = 1.0 / (dbl(B * Tn) * pi)
    else:
        C = torch.minimum(torch.full_like(T, max(case["C"], 1)), T)
        x, _, _, _ = _philox(zero(ids), ids, torch.ones_like(ids), torch.full_like(ids, 3), key0, key1)
        cut = T.clone()
        cut = torch.where(scheme == nat.RPC, C + ((x * (T - C + 1)) >> 32), cut)
        cut = torch.where(scheme == nat.DET, torch.floor(0.5 * dbl(T)).long(), cut)
        keep = t0 < cut[seq]
        p = torch.ones(N, dtype=torch.float64, device=DEV)
        if case["scheme"] in ("urs", "mixed"):
            urs = scheme[seq] == nat.URS
            keep = torch.where(urs, word < int(math.floor(case["p"] * 4294967296.0)), keep)
            p = torch.where(urs, torch.full_like(p, case["p"]), p)
        if case["scheme"] == "rpc":
            p = torch.where(t0 + 1 > C[seq], dbl(Tn - t0) / dbl(Tn - C[seq] + 1), p)
        w = 1.0 / (dbl(B * Tn) * p)
    if adv is not None:
        keep = keep & (adv[seq] != 0)
    k = torch.nonzero(keep)[:, 0]
    return k, seq[k], w[k], pi


def _exact_loss(hidden, W, ids, old, A, w, ref=None, kl="none", beta=0.0, dW=None):
    """The loss stage in 64 bits on the GPU, token block by token block."""
    n, V = hidden.shape[0], W.shape[0]
    W64 = W.double()
    if dW is None:
        dW = torch.zeros_like(W64)
    o = dict(logp=torch.empty(n, dtype=torch.float64, device=DEV), kl=torch.zeros(n, dtype=torch.float64, device=DEV),
             entropy=torch.empty(n, dtype=torch.float64, device=DEV),
             dH=torch.empty(hidden.shape, dtype=torch.float64, device=DEV), dW=dW)
    loss = torch.zeros((), dtype=torch.float64, device=DEV)
    for k0 in range(0, n, 4096):
        k = slice(k0, min(n, k0 + 4096))
        h, y = hidden[k].double(), ids[k].long()
        z = h @ W64.t()
        lse = torch.logsumexp(z, 1)
        logp = z.gather(1, y[:, None])[:, 0] - lse
        prob = torch.exp(z - lse[:, None])
        o["logp"][k], o["entropy"][k] = logp, lse - (prob * z).sum(1)
        r, a = torch.exp(logp - old[k].double()), A[k].double()
        S = torch.minimum(r * a, r.clamp(1 - 0.2, 1 + 0.2) * a)
        active = ((a > 0) & (r <= 1 + 0.2)) | ((a < 0) & (r >= 1 - 0.2))
        g = torch.where(active, r * a, torch.zeros_like(a))
        if kl != "none":
            d = ref[k].double() - logp
            term, slope = (torch.exp(d) - d - 1, 1 - torch.exp(d)) if kl == "nonneg" else (-d, torch.ones_like(d))
            o["kl"][k] = term
            S, g = S - beta * term, g - beta * slope
        loss -= (w[k].double() * S).sum()
        c = -w[k].double() * g
        dz = prob.mul_(-c[:, None])
        dz[torch.arange(dz.shape[0], device=DEV), y] += c
        o["dH"][k] = dz @ W64
        dW += dz.t() @ h
        del z, prob, dz
    o["loss"] = loss.reshape(1)
    return o


def exact(case, seed):
    if case["kind"] != "select" and work(case)["flops"] > 1.2e14:
        return None
    s = prepare(case, seed)
    if case["kind"] == "select":
        k, seq, w, pi = _exact_selection(s)
        kept_w = torch.zeros(max(s["N"], 1), dtype=torch.float64, device=DEV)
        kept_w[:len(k)] = w
        out = dict(kept_w=kept_w)
        if case["scheme"] == "schedule" and s["N"] > 0:
            out["pi"] = pi
        return out
    if case["kind"] == "logp":
        n = case["tokens"]
        logp, ent = (torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(2))
        W64 = s["W"].double()
        for k0 in range(0, n, 4096):
            k = slice(k0, min(n, k0 + 4096))
            z = s["hidden"][k].double() @ W64.t()
            lse = torch.logsumexp(z, 1)
            logp[k] = z.gather(1, s["ids"][k].long()[:, None])[:, 0] - lse
            if case["entropy"]:
                ent[k] = lse - (torch.exp(z - lse[:, None]) * z).sum(1)
        return dict(logp=logp, entropy=ent if case["entropy"] else None)
    if case["kind"] == "step":
        R = torch.from_numpy(s["R"]).to(DEV).double()
        adv = ((R - R.mean(1, keepdim=True)) / (R.std(1, unbiased=False, keepdim=True) + 1e-6)).reshape(-1)
        k, seq, w, _ = _exact_selection(s, adv if case["drop"] else None)
        o = _exact_loss(s["hidden"][k], s["W"], s["ids"][k], s["old_logp"][k], adv[seq], w)
        return dict(adv=adv, kept_idx=None, kept_w=w, loss=o["loss"], logp=o["logp"], dH=o["dH"], dW=o["dW"])
    parts, dW, n = [], None, case["tokens"]
    for m in range(case["micro"]):
        k = slice(m * n, (m + 1) * n)
        o = _exact_loss(s["hidden"][k], s["W"], s["ids"][k], s["old_logp"][k], s["adv"][s["kept_seq"][k].long()],
                        s["kept_w"][k], s["ref_logp"][k] if case["kl"] != "none" else None, case["kl"], 0.04, dW)
        dW = o["dW"]
        parts.append(dict(loss=o["loss"], logp=o["logp"], dH=o["dH"], kl=o["kl"] if case["kl"] != "none" else None,
                          entropy=o["entropy"] if case["entropy"] else None))
    return dict(parts=parts, dW=dW)
