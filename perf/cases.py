"""What the performance of this library is measured on.

Every case is one call of a public entry point of `paper_2602_19362_amd.oapl`, on buffers that a
trainer or a rollout harness has in hand: hidden states and LM-head weights in device memory, a
workspace (and gradient buffers) allocated once and reused from step to step.  The kinds of call:

    loss      loss_fwd_bwd, gradients included: the trainer step
    loss_fwd  loss_fwd_bwd without gradients: evaluating the objective on a held-out batch
    grpo      grpo_loss_fwd_bwd, gradients included: the baseline objective on the same head
    score     logprob_fwd: log-probs (and log-sum-exp, policy entropy) of sampled tokens
    sample    sample_tokens: one draw per row, from one decode step's rows to whole blocks

Hidden states are unit Gaussians with a share of the sampled token's own weight row mixed in, so
that sampled tokens range from unlikely to near-certain as a trained policy's do (pure Gaussian
rows would give every token a log-prob near -ln V).  Weights are N(0, 1/d), rollout lengths are
lognormal (sigma 0.6) scaled to the case's token count and cut at the generation limit, rewards are
0/1, and the inference policy's log-probs are the current ones (to the accuracy of a Gaussian
estimate of the log-sum-exp) plus a drift of standard deviation 0.1.
"""
import math

import numpy as np
import torch

from paper_2602_19362_amd import oapl

DEVICE = "cuda:0"
VOCAB = 151936            # the vocabulary of every bf16 configuration of this repository


def _loss(name, dtype, d, V, T, prompts, rollouts, cap, **kw):
    c = {"kind": "loss", "dtype": dtype, "d": d, "V": V, "T": T, "prompts": prompts, "rollouts": rollouts, "cap": cap,
         "beta": 0.5}
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the exactness configuration: two prompts x four rollouts of 32 tokens in fp32; a call that is all latency
        _loss("loss_f32_tiny", "f32", 64, 1024, 256, 2, 4, 32, beta=1.0),
        # fp32 used in earnest: checking a bf16 training run's head against full precision on a small policy
        _loss("loss_f32_small_policy", "f32", 768, 8192, 1501, 2, 4, 512, beta=1.0),
        # a debugging-size policy in bf16 (the head of the smoke check), through the entry point that allocates nothing
        _loss("loss_bf16_small_head", "bf16", 256, 1544, 1000, 2, 4, 400, noalloc=True),
        # one decode step of eight prompts x eight rollouts at the 7B-class head
        {"name": "sample_decode_step", "kind": "sample", "dtype": "bf16", "d": 4096, "V": VOCAB, "T": 64,
         "temperature": 1.0},
        # draws for whole blocks of positions (how the 1.7B-class workload draws its tokens)
        {"name": "sample_block", "kind": "sample", "dtype": "bf16", "d": 2048, "V": VOCAB, "T": 4096,
         "temperature": 0.8},
        # rescoring one short rollout with its log-sum-exp and entropy (monitoring while a run goes on)
        {"name": "score_one_rollout_entropy", "kind": "score", "dtype": "bf16", "d": 4096, "V": VOCAB, "T": 777,
         "lse": True, "entropy": True},
        # the forward-only workload: four prompts x eight rollouts of 1024 tokens at the 1.7B-class head
        {"name": "score_batch", "kind": "score", "dtype": "bf16", "d": 2048, "V": VOCAB, "T": 32768, "lse": False,
         "entropy": False},
        # a micro-batch of one prompt whose eight answers are short
        _loss("loss_short_answers", "bf16", 4096, VOCAB, 1003, 1, 8, 512),
        # one prompt's eight answers at the math workload's lengths, baseline objective, 1.7B-class head
        {"name": "grpo_one_prompt", "kind": "grpo", "dtype": "bf16", "d": 2048, "V": VOCAB, "T": 6007, "prompts": 1,
         "rollouts": 8, "cap": 4096},
        # one prompt's eight answers, 7B-class head, two betas as in the experiments
        _loss("loss_one_prompt", "bf16", 4096, VOCAB, 16411, 1, 8, 4096, beta=1.0, beta_value=0.25),
        # long code rollouts at the 14B-class head: lengths up to 16384, a ring of panel buffers
        _loss("loss_long_rollouts", "bf16", 5120, VOCAB, 30011, 1, 4, 16384, beta=1.0),
        # the benchmark batch: eight prompts x eight rollouts, T as its length law draws it
        _loss("loss_full_batch", "bf16", 4096, VOCAB, 140897, 8, 8, 4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loss", "loss", "loss", "loss_fwd", "grpo", "score", "score", "sample", "sample", "loss_f32",
                       "loss_small"])
    if kind == "loss_f32":
        T = _log_int(rng, 32, 2000)
        prompts = rng.randint(1, 3)
        return _loss(None, "f32", rng.randint(16, 768), _log_int(rng, 500, 8192), T, prompts, rng.randint(2, 6),
                     max(32, T), beta=1.0)
    if kind == "loss_small":
        T = _log_int(rng, 64, 1000)
        return _loss(None, "bf16", 8 * rng.randint(8, 32), _log_int(rng, 300, 1544), T, rng.randint(1, 3), 4,
                     max(32, T), noalloc=True)
    # heads of language-model size: hidden sizes of the configurations and odd multiples of eight between them
    d = rng.choice([1024, 2048, 4096, 5120, 8 * rng.randint(128, 640)])
    V = rng.choice([VOCAB, VOCAB, _log_int(rng, 32000, VOCAB)])
    if kind == "sample":
        return {"kind": "sample", "dtype": "bf16", "d": d, "V": V, "T": _log_int(rng, 1, 8192),
                "temperature": rng.choice([0.6, 0.8, 1.0, 1.2])}
    if kind == "score":
        return {"kind": "score", "dtype": "bf16", "d": d, "V": V, "T": _log_int(rng, 8, 32768),
                "lse": rng.random() < 0.5, "entropy": rng.random() < 0.5}
    prompts, rollouts = rng.choice([1, 1, 2, 4]), rng.choice([4, 8])
    T = _log_int(rng, 100, 48000)
    cap = 4 * (T // (prompts * rollouts) + 1)
    if kind == "grpo":
        return {"kind": "grpo", "dtype": "bf16", "d": d, "V": V, "T": T, "prompts": prompts, "rollouts": rollouts,
                "cap": cap}
    c = _loss(None, "bf16", d, V, T, prompts, rollouts, cap, beta=rng.choice([0.5, 1.0, 2.0]))
    c["kind"] = kind
    if rng.random() < 0.3:
        c["beta_value"] = 0.25
    return c


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _randn(rows, cols, std, dtype, gen):
    """N(0, std^2), drawn in fp32 slab by slab and rounded once."""
    out = torch.empty((rows, cols), dtype=dtype, device=DEVICE)
    slab = max(1, (1 << 27) // cols)
    for r0 in range(0, rows, slab):
        r1 = min(rows, r0 + slab)
        out[r0:r1] = (torch.randn((r1 - r0, cols), generator=gen, device=DEVICE) * std).to(dtype)
    return out


def _lengths(case, seed):
    """Rollout lengths: lognormal shares of T, each at most the generation limit, summing to T."""
    n, T, cap = case["prompts"] * case["rollouts"], case["T"], case["cap"]
    assert n * cap >= T
    rng = np.random.default_rng(seed)
    share = np.exp(0.6 * rng.standard_normal(n))
    lens = np.minimum(np.floor(T * share / share.sum()).astype(np.int64), cap)
    while lens.sum() < T:                       # what the cut and the rounding left over goes to the others
        room = cap - lens
        left = T - int(lens.sum())
        add = np.minimum(room, np.maximum(1, left * room // max(1, int(room.sum()))))
        add = np.minimum(add, np.maximum(0, left - (np.cumsum(add) - add)))
        lens = lens + add
    return lens


def prepare(case, seed):
    dt, d, V, T = _dtype(case), case["d"], case["V"], case["T"]
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    code = oapl.OAPL_F32 if case["dtype"] == "f32" else oapl.OAPL_BF16
    W = _randn(V, d, 1.0 / math.sqrt(d), dt, gen)
    tokens = torch.randint(0, V, (T,), generator=gen, device=DEVICE, dtype=torch.int64).to(torch.int32)
    H = torch.empty((T, d), dtype=dt, device=DEVICE)
    zy = torch.empty(T, device=DEVICE)
    half_var = torch.empty(T, device=DEVICE)
    slab = max(1, (1 << 26) // d)
    for r0 in range(0, T, slab):
        r1 = min(T, r0 + slab)
        w = W[tokens[r0:r1].long()].float()
        pull = 16.0 * torch.rand((r1 - r0, 1), generator=gen, device=DEVICE)     # sampled token's logit: 0 .. 16
        h = (torch.randn((r1 - r0, d), generator=gen, device=DEVICE) + pull * w).to(dt)
        H[r0:r1] = h
        h = h.float()
        zy[r0:r1] = (h * w).sum(1)
        half_var[r0:r1] = (h * h).sum(1) / (2.0 * d)
    state = {"case": case, "H": H, "W": W, "tokens": tokens, "code": code}
    if case["kind"] in ("sample", "score"):
        nbytes = oapl.workspace_bytes(T, d, V, 0, 1, code, False)
        state["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)
        state["draw_seed"] = seed
        return state

    n_seq = case["prompts"] * case["rollouts"]
    lens = _lengths(case, seed)
    off = np.zeros(n_seq + 1, dtype=np.int64)
    off[1:] = np.cumsum(lens)
    lp = zy - torch.logaddexp(zy, half_var + math.log(V))
    noise = torch.randn(T, generator=gen, device=DEVICE)
    state["logq"] = torch.clamp(lp + 0.1 * noise, max=0.0).contiguous()
    state["off"] = torch.from_numpy(off).to(DEVICE)
    state["rewards"] = (torch.rand(n_seq, generator=gen, device=DEVICE) < 0.4).float()
    state["gid"] = (torch.arange(n_seq, device=DEVICE) // case["rollouts"]).to(torch.int32)
    backward = case["kind"] != "loss_fwd"
    if case["kind"] == "grpo":
        state["logp_old"] = (lp + 0.05 * torch.randn(T, generator=gen, device=DEVICE)).contiguous()
    if backward:
        state["dH"] = torch.empty_like(H)
        state["dW"] = torch.empty((V, d), dtype=torch.float32, device=DEVICE)
    if case.get("noalloc"):
        state["loss"] = torch.empty(1, device=DEVICE)
        state["logprob"] = torch.empty(T, device=DEVICE)
        state["ratio"] = torch.empty(n_seq, device=DEVICE)
        state["vstar"] = torch.empty(case["prompts"], device=DEVICE)
    else:
        nbytes = oapl.workspace_bytes(T, d, V, n_seq, case["prompts"], code, backward, max_rollout_len=case["cap"])
        state["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    case, s = state["case"], state
    kind = case["kind"]
    if kind == "sample":
        tok, score, _ = oapl.sample_tokens(s["H"], s["W"], case["temperature"], s["draw_seed"], want_scores=True,
                                           workspace=s["workspace"])
        return {"tokens": tok, "scores": score}
    if kind == "score":
        out = oapl.logprob_fwd(s["H"], s["W"], s["tokens"], want_lse=case["lse"], want_entropy=case["entropy"],
                               workspace=s["workspace"])
        return list(out[:-1])
    if kind == "grpo":
        r = oapl.grpo_loss_fwd_bwd(s["H"], s["W"], s["tokens"], s["logq"], s["logp_old"], s["off"], s["rewards"],
                                   s["gid"], case["prompts"], workspace=s["workspace"], dH=s["dH"], dW=s["dW"])
        return {"loss": r.loss, "logprob": r.logprob, "advantages": r.advantages, "dH": r.dH, "dW": r.dW}
    if case.get("noalloc"):
        oapl.loss_fwd_bwd_noalloc(s["H"], s["W"], s["tokens"], s["logq"], s["off"], s["rewards"], s["gid"],
                                  case["prompts"], case["beta"], s["loss"], s["logprob"], s["ratio"], s["vstar"],
                                  s["dH"], s["dW"])
        return {k: s[k] for k in ("loss", "logprob", "ratio", "vstar", "dH", "dW")}
    r = oapl.loss_fwd_bwd(s["H"], s["W"], s["tokens"], s["logq"], s["off"], s["rewards"], s["gid"], case["prompts"],
                          case["beta"], beta_value=case.get("beta_value"), backward=kind == "loss",
                          workspace=s["workspace"], dH=s.get("dH"), dW=s.get("dW"))
    out = {"loss": r.loss, "logprob": r.logprob, "ratio": r.seq_logratio, "vstar": r.vstar}
    if kind == "loss":
        out.update(dH=r.dH, dW=r.dW)
    return out


def work(case):
    d, V, T = case["d"], case["V"], case["T"]
    e = 4 if case["dtype"] == "f32" else 2
    gemm = 2.0 * T * V * d                                   # one T x V x d contraction
    bytes_ = e * (T * d + V * d)                             # hidden states and weights, once each
    if case["kind"] == "sample":
        return {"bytes": bytes_ + 8 * T, "flops": gemm}      # tokens and scores out
    if case["kind"] == "score":
        return {"bytes": bytes_ + 8 * T + 4 * T * (int(case["lse"]) + int(case["entropy"])), "flops": gemm}
    bytes_ += 12 * T                                         # tokens and inference log-probs in, log-probs out
    if case["kind"] == "loss_fwd":
        return {"bytes": bytes_, "flops": gemm}
    if case["kind"] == "grpo":
        bytes_ += 4 * T
    return {"bytes": bytes_ + e * T * d + 4 * V * d, "flops": 3 * gemm}      # dH and dW out


def tolerance(case):
    """About four times what the outputs differ from the same formulas in fp64 (largest over the outputs)."""
    if case["kind"] == "sample":
        # scores carry fp32 logits and logarithms; a draw may change only where its two best scores tie in fp32
        return {"rel": 3e-6, "differ": 1e-3}
    if case["kind"] == "score":
        return {"rel": 3e-6}                # fp32 sums of exact bf16 products: 2e-7 .. 6e-7 seen
    if case["dtype"] == "f32":
        return {"rel": 1e-4}                # residuals are differences of sums over a rollout: 5e-6 .. 2.5e-5 seen
    if case["kind"] == "loss_fwd":
        return {"rel": 2e-4}                # the same residuals, squared in the loss: 1e-5 .. 6e-5 seen
    return {"rel": 7e-3}                    # bf16 roundings of the soft-max panel, scaled rows and dH: 1.7e-3 seen
