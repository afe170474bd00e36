"""The work that a user of this library has it do, as a list of timed cases and a generator of more of the same kinds.

A training step of AIS-GRPO calls the library in one of three ways: on materialised trainer logits with the three-call
path (`AisContext.step`), on materialised logits with each row read once (`AisContext.step_one_sweep`), or on the last
hidden states and the output embedding (`lm_head_logprob`, `diagnostics`, `grpo_row_scale`, `lm_head_grad`).  The
rollout side adds the FP8 perturbation of logits.  Every case is one such call or chain of calls through
`paper_2605_13907_amd.binding.AisContext`, on synthetic inputs of the shapes and value distributions of
`paper_2605_13907_amd.workloads`.

Kinds (the `kind` of a case):
  step         the three-call path: log-probs, diagnostics and alpha, loss and gradient w.r.t. the logits
  one_sweep    log-probs and unscaled gradient direction in one sweep, diagnostics, per-row scale
  fp8_logprob  log-prob of the sampled tokens under the FP8-E4M3 round trip of the logits
  fp8_codes    FP8-E4M3 codes and scales of the logits, and their decoding back to the logits' type
  head_logprob log-probs from hidden states and output embedding, no gradient (the old-policy / reference pass)
  head_step    the whole step from hidden states: log-probs, diagnostics, per-row scale, both gradients
  scalars      diagnostics and per-row scale alone, on log-probs that the trainer has already (a global batch)

Layouts: `packed` responses follow each other without padding; `padded` every response owns rows / responses rows and
uses the first part of them; `masked` (masked diffusion) a random subset of every response's rows is evaluated.
"""
import functools
import math

import torch

from paper_2605_13907_amd import binding, workloads

E4M3_MAX = 448.0


def listed():
    return [
        # Launch latency: a debugging or smoke-test step (workload 1 of the benchmark).
        dict(name="step-tiny-f32", kind="step", rows=512, vocab=1024, dtype="f32", responses=8, group=4,
             layout="padded", stale=False),
        # The flagship: one training step on two prompts' worth of rollouts (workload 2 of the benchmark, full size).
        dict(name="step-packed-bf16", kind="step", rows=41_643, vocab=151_936, dtype="bf16", responses=16, group=8,
             layout="packed", stale=False),
        # Masked-diffusion rollouts (workload 3's shape, a quarter of its responses): half of the rows are evaluated.
        dict(name="step-masked-bf16", kind="step", rows=8_192, vocab=126_464, dtype="bf16", responses=16, group=8,
             layout="masked", stale=False),
        # A later optimisation step on the same rollouts (stale policy, KL term, rollout temperature) with a vocabulary
        # that is not a multiple of anything: a contiguous [rows, vocab] tensor as a plain read-out layer returns it.
        dict(name="step-odd-vocab-stale-bf16", kind="step", rows=12_345, vocab=50_257, dtype="bf16", responses=32,
             group=8, layout="packed", stale=True),
        # fp32 logits, the other storage type, with an odd vocabulary and padded responses.
        dict(name="step-odd-vocab-f32", kind="step", rows=4_096, vocab=32_003, dtype="f32", responses=16, group=4,
             layout="padded", stale=False),
        # The widest vocabulary (workload 4's), each row read once.
        dict(name="one-sweep-wide-bf16", kind="one_sweep", rows=8_411, vocab=248_320, dtype="bf16", responses=32,
             group=8, layout="packed", stale=False),
        # The sampler's side of the ratio for a batch of rollouts.
        dict(name="fp8-logprob-bf16", kind="fp8_logprob", rows=10_411, vocab=151_936, dtype="bf16", responses=8,
             group=8, layout="packed", stale=False),
        # The low-precision logits themselves, there and back.
        dict(name="fp8-codes-bf16", kind="fp8_codes", rows=8_192, vocab=126_464, dtype="bf16", responses=16, group=8,
             layout="packed", stale=False),
        # One short prompt group scored from hidden states: the output embedding is most of what is read.
        dict(name="head-logprob-short", kind="head_logprob", rows=390, vocab=151_936, d_model=4_096, responses=8,
             group=8, layout="packed", stale=False),
        # The no-gradient pass over a whole training batch of the flagship workload.
        dict(name="head-logprob-long", kind="head_logprob", rows=41_643, vocab=151_936, d_model=4_096, responses=16,
             group=8, layout="packed", stale=False),
        # The whole masked-diffusion step without materialised logits.
        dict(name="head-step-masked", kind="head_step", rows=8_192, vocab=126_464, d_model=4_096, responses=16,
             group=8, layout="masked", stale=False),
        # Correction of a global batch whose log-probs come from elsewhere.
        dict(name="scalars-global-batch", kind="scalars", rows=1_200_000, vocab=0, dtype="f32", responses=1_024,
             group=8, layout="packed", stale=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["step", "step", "step", "one_sweep", "one_sweep", "fp8_logprob", "fp8_codes", "head_logprob",
                       "head_step", "scalars"])
    group = rng.choice([4, 8])
    responses = group * log_int(1, 16)
    layout = rng.choice(["packed", "packed", "padded", "masked"])
    stale = rng.random() < 0.3
    if kind == "scalars":
        responses = group * log_int(1, 512)
        return dict(kind=kind, rows=log_int(20_000, 4_000_000), vocab=0, dtype="f32", responses=responses, group=group,
                    layout="packed", stale=stale)
    # vocabularies from a byte-level model's to the widest; most are padded to a multiple of 64, some are what they are
    vocab = log_int(1_000, 262_144)
    if rng.random() < 0.6:
        vocab = max(64, vocab // 64 * 64)
    if kind in ("head_logprob", "head_step"):
        d_model = 64 * log_int(8, 80)
        rows = log_int(200, 20_000)
        rows = min(rows, max(64, int(1.5e13 / (6.0 * vocab * d_model))))
        rows = -(-rows // responses) * responses + (rng.randrange(responses) if layout == "packed" else 0)
        return dict(kind=kind, rows=rows, vocab=vocab, d_model=d_model, responses=responses, group=group,
                    layout=layout, stale=False)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    rows = min(log_int(200, 60_000), max(64, int((1.2e9 if dtype == "bf16" else 0.6e9) / vocab)))
    rows = -(-rows // responses) * responses + (rng.randrange(responses) if layout == "packed" else 0)
    return dict(kind=kind, rows=rows, vocab=vocab, dtype=dtype, responses=responses, group=group, layout=layout,
                stale=stale)


# ---- inputs ----------------------------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def context():
    """The one context that a program keeps."""
    return binding.AisContext()


def structure(case):
    """(row offsets [B + 1], used rows of each response [B]) as lists: what the case alone decides."""
    n, b = case["rows"], case["responses"]
    share = [0.25 + 0.75 * ((i + 1) * 0.6180339887 % 1.0) for i in range(b)]
    if case["layout"] == "packed":
        total, run, offsets = sum(share), 0.0, [0]
        for s in share:
            run += s
            offsets.append(int(round(n * run / total)))
        offsets[-1] = n
        return offsets, [offsets[i + 1] - offsets[i] for i in range(b)]
    pitch = n // b
    return [i * pitch for i in range(b + 1)], [max(1, int(pitch * s)) for s in share]


def valid_rows(case):
    """Number of evaluated rows (its expectation for masked layouts)."""
    offsets, used = structure(case)
    if case["layout"] == "masked":
        return case["rows"] // 2
    return sum(used)


def valid_mask(case, gen):
    """[rows] uint8 on the GPU, or None where every row is evaluated."""
    if case["layout"] == "packed":
        return None
    b, pitch = case["responses"], case["rows"] // case["responses"]
    if case["layout"] == "padded":
        used = torch.tensor(structure(case)[1], device="cuda")
        mask = torch.arange(pitch, device="cuda").unsqueeze(0) < used.unsqueeze(1)
    else:                       # the mask ratio of a diffusion step is uniform: here one value of each b-th part
        ratio = (torch.arange(b, device="cuda", dtype=torch.float32) + 0.5) / b
        mask = torch.rand(b, pitch, generator=gen, device="cuda") < ratio.unsqueeze(1)
    return mask.to(torch.uint8).reshape(-1).contiguous()


def rewards_of(case, gen):
    """0 / 1 rewards; no prompt's responses are all equal (such prompts are usually filtered out)."""
    b = case["responses"]
    r = (torch.rand(b, generator=gen, device="cuda") < 0.4).to(torch.float32)
    r[0::case["group"]] = 1.0
    r[1::case["group"]] = 0.0
    return r


def params_of(case):
    if case["stale"]:
        return binding.default_params(beta_kl=0.04, inv_temperature=1.0 / 0.9)
    return binding.default_params()


def make_logits(case, gen):
    """Trainer logits, the tokens an FP8 sampler drew, and the sampler's log-probs of them (noise on top, as between
    two engines): [rows, vocab], [rows] int32, [rows] fp32."""
    n, v = case["rows"], case["vocab"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    logits = torch.empty(n, v, dtype=dt, device="cuda")
    tokens = torch.empty(n, dtype=torch.int32, device="cuda")
    logp = torch.empty(n, dtype=torch.float32, device="cuda")
    step = max(1, int(1.5e8) // v)
    for r0 in range(0, n, step):
        z = torch.randn(min(step, n - r0), v, generator=gen, device="cuda") * 3.0
        top = z.argmax(dim=1, keepdim=True)
        boost = 8.0 * torch.rand(z.shape[0], 1, generator=gen, device="cuda")     # from flat to peaked rows
        z.scatter_add_(1, top, boost)
        logits[r0:r0 + step] = z.to(dt)
        z = workloads.fp8_rollout_logits(logits[r0:r0 + step].float())
        z += torch.randn(z.shape, generator=gen, device="cuda") * 0.5
        gumbel = torch.rand(z.shape, generator=gen, device="cuda").clamp_(min=1e-38).log_().neg_().log_().neg_()
        y = (z + gumbel).argmax(dim=1, keepdim=True)
        tokens[r0:r0 + step] = y.squeeze(1).to(torch.int32)
        logp[r0:r0 + step] = (z.gather(1, y) - torch.logsumexp(z, dim=1, keepdim=True)).squeeze(1)
    return logits, tokens, logp


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * (seed % 1_000_000) + 17)
    n, b, kind = case["rows"], case["responses"], case["kind"]
    s = dict(case=case, ctx=context(), params=params_of(case), valid=valid_mask(case, gen), rewards=rewards_of(case, gen),
             cu_rows=torch.tensor(structure(case)[0], dtype=torch.int64, device="cuda"), logp_old=None, logp_ref=None)
    if kind == "scalars":
        s["logp"] = -torch.rand(n, generator=gen, device="cuda").mul_(8.0).square_().div_(8.0)
        s["logp_roll"] = (s["logp"] + 0.3 * torch.randn(n, generator=gen, device="cuda")).clamp_(max=0.0)
    elif kind in ("head_logprob", "head_step"):
        v, d = case["vocab"], case["d_model"]
        w = torch.empty(v, d, dtype=torch.bfloat16, device="cuda")
        for v0 in range(0, v, 32_768):
            w[v0:v0 + 32_768] = (torch.randn(min(32_768, v - v0), d, generator=gen, device="cuda") / math.sqrt(d)).bfloat16()
        # every row prefers one token, from nearly flat to sharply peaked; that token is sampled with probability 0.7
        mode = torch.randint(0, v, (n,), generator=gen, device="cuda")
        sharp = 12.0 * torch.rand(n, 1, generator=gen, device="cuda")
        wm = w[mode].float()
        noise = torch.randn(n, d, generator=gen, device="cuda")
        s["hidden"] = (sharp * wm / (wm * wm).sum(dim=1, keepdim=True).clamp_min(1e-6) + noise).bfloat16()
        other = torch.randint(0, v, (n,), generator=gen, device="cuda")
        pick = torch.rand(n, generator=gen, device="cuda") < 0.7
        s["weight"] = w
        s["tokens"] = torch.where(pick, mode, other).to(torch.int32)
        # the sampler's log-prob: near what a row of this sharpness gives its token
        own = (s["hidden"].float() * w[s["tokens"].long()].float()).sum(dim=1)
        lse = torch.logaddexp(sharp.squeeze(1), torch.full((n,), math.log(v) + 0.5, device="cuda"))
        s["logp_roll"] = (own - lse + 0.5 * torch.randn(n, generator=gen, device="cuda")).clamp_(max=-1e-4).contiguous()
        # a diffusion loader knows how many positions it masked
        s["n_live"] = -1 if s["valid"] is None else int(s["valid"].sum().item())
    else:
        s["logits"], s["tokens"], s["logp_roll"] = make_logits(case, gen)
        if kind in ("step", "one_sweep"):
            shape = workloads.RolloutShape("case", b // case["group"], case["group"], case["vocab"], case["dtype"], 3.0,
                                           0.0, "packed", n, ("fixed",), 0.4)
            s["batch"] = workloads.RolloutBatch(shape, s["logits"], s["tokens"], s["valid"], s["cu_rows"],
                                                s["logp_roll"], s["rewards"], torch.tensor(structure(case)[1]))
    if s["valid"] is not None:
        off = s["valid"] == 0
        s["logp_roll"][off] = 0.0
        if "tokens" in s:
            s["tokens"][off] = -1
    if case["stale"]:            # the policy one update ago and a reference policy, near the sampler's log-probs
        base = s["logp"] if kind == "scalars" else s["logp_roll"]
        s["logp_old"] = (base + 0.05 * torch.randn(n, generator=gen, device="cuda")).clamp_(max=0.0)
        s["logp_ref"] = (base + 0.10 * torch.randn(n, generator=gen, device="cuda")).clamp_(max=0.0)
    return s


# ---- one pass ------------------------------------------------------------------------------------------------------

def diag_values(diag):
    """The fifteen fp64 statistics of the device ais_diag (mean_w ... mean_abs_dp)."""
    return diag[8:128].view(torch.float64)


def run(s):
    ctx, case, p = s["ctx"], s["case"], s["params"]
    kind = case["kind"]
    if kind in ("step", "one_sweep"):
        step = ctx.step if kind == "step" else ctx.step_one_sweep
        out = step(s["batch"], p, s["logp_old"], s["logp_ref"])
        out["diag"] = diag_values(out["diag"])
        return out
    if kind == "fp8_logprob":
        return ctx.fp8_rollout_logprob(s["logits"], s["tokens"], s["valid"])
    if kind == "fp8_codes":
        codes, scale = ctx.fp8_quantize_rows(s["logits"])
        return dict(codes=codes, scale=scale, z=ctx.fp8_dequantize_rows(codes, scale, s["logits"].dtype))
    if kind == "scalars":
        adv, count, diag = ctx.diagnostics(s["logp"] if s["logp_old"] is None else s["logp_old"], s["logp_roll"],
                                           s["valid"], s["cu_rows"], s["rewards"], case["group"], p)
        loss, wtilde, g = ctx.grpo_row_scale(s["logp"], s["logp_roll"], s["valid"], s["cu_rows"], adv, count, diag, p,
                                             s["logp_old"], s["logp_ref"])
        return dict(adv=adv, count=count, diag=diag_values(diag), loss=loss, wtilde=wtilde, g=g)
    logp, lse = ctx.lm_head_logprob(s["hidden"], s["weight"], s["tokens"], s["valid"], p.inv_temperature)
    if kind == "head_logprob":
        return dict(logp=logp, lse=lse)
    adv, count, diag = ctx.diagnostics(logp, s["logp_roll"], s["valid"], s["cu_rows"], s["rewards"], case["group"], p)
    loss, wtilde, g = ctx.grpo_row_scale(logp, s["logp_roll"], s["valid"], s["cu_rows"], adv, count, diag, p)
    dh, dw = ctx.lm_head_grad(s["hidden"], s["weight"], s["tokens"], lse, logp, g, p.inv_temperature,
                              n_live_max=s["n_live"])
    return dict(logp=logp, lse=lse, adv=adv, count=count, diag=diag_values(diag), loss=loss, wtilde=wtilde, g=g,
                dhidden=dh, dweight=dw)


def work(case):
    n, v, kind = case["rows"], case["vocab"], case["kind"]
    live = valid_rows(case)
    per_row = 4 * (5 + (2 if case["stale"] else 0)) + 1      # token, logp, lse, logp_roll, wtilde, ... and the mask
    if kind == "scalars":
        return dict(bytes=n * 4.0 * (4 + (2 if case["stale"] else 0)), flops=40.0 * n)
    if kind in ("head_logprob", "head_step"):
        d = case["d_model"]
        once = 2.0 * (live * d + v * d)
        if kind == "head_logprob":
            return dict(bytes=once + per_row * n, flops=2.0 * live * v * d)
        # the logits, and the two products that their gradient enters
        return dict(bytes=once + 4.0 * (n * d + v * d) + per_row * n, flops=6.0 * live * v * d)
    e = 2.0 if case["dtype"] == "bf16" else 4.0
    if kind == "fp8_logprob":
        return dict(bytes=e * live * v + 9 * n, flops=4.0 * live * v)
    if kind == "fp8_codes":
        return dict(bytes=2 * e * n * v + n * v + 4 * n, flops=4.0 * n * v)
    return dict(bytes=e * v * (live + n) + per_row * n, flops=8.0 * live * v)


def tolerance(case):
    """Measured against 64 bits (`exact`): log-probs 2e-7, statistics and weights 1e-7 to 2e-6, bf16 gradients 2e-3,
    the products of bf16 gradients 2e-3; the loss, a difference of near-equal sums of fp32 log-probs, up to 2e-5."""
    kind = case["kind"]
    if kind == "fp8_codes":
        return "exact"              # codes are bytes; scale and decoded value are one correctly rounded operation each
    if kind == "head_step":
        return {"rel": 4e-3, "max": 0.3}      # dlogits are rounded to bf16 before the products
    if kind in ("step", "one_sweep"):
        # a bf16 rounding that falls the other way is 2^-8 of the element
        return {"rel": 4e-3, "max": 0.02} if case["dtype"] == "bf16" else {"rel": 1e-4, "max": 2e-3}
    return {"rel": 1e-6, "max": 1e-4}         # fp32 log-probs and weights


# ---- the same in 64 bits ---------------------------------------------------------------------------------------------

def exact_scalars(s, logp, logp_old, logp_ref):
    """Ratios, diagnostics, alpha, weights, loss and per-row coefficient from fp64 log-probs (Eq. 3, 10, 12-19)."""
    case, p = s["case"], s["params"]
    n, b = case["rows"], case["responses"]
    c, delta, gamma, eps, beta = 5.0, float(torch.tensor(0.02)), float(torch.tensor(1.2)), float(torch.tensor(1e-6)), 1.0
    valid = torch.ones(n, dtype=torch.bool, device="cuda") if s["valid"] is None else s["valid"].bool()
    cu = s["cu_rows"]
    resp = torch.repeat_interleave(torch.arange(b, device="cuda"), cu[1:] - cu[:-1])
    count = torch.zeros(b, dtype=torch.float64, device="cuda").index_add_(0, resp, valid.double())
    old = logp if logp_old is None else logp_old
    roll = s["logp_roll"].double()
    d = (old - roll)[valid]
    w = d.clamp(max=math.log(c)).exp()
    rw = s["rewards"].double().view(-1, case["group"])
    adv = (rw - rw.mean(dim=1, keepdim=True)).reshape(-1)
    a32 = adv.float().double()
    a = a32[resp][valid]
    mean_w, var_w = w.mean(), w.var(unbiased=False)
    cv2 = var_w / mean_w ** 2
    dbar, std_a, std_aw = d.abs().mean(), a.std(unbiased=False), (a * w).std(unbiased=False)
    dsigma = std_aw / (std_a + eps)
    a_ess, a_mis = (1 + cv2) ** -0.5, (dbar / delta).clamp(max=1.0)
    a_var = ((dsigma - gamma) / gamma).clamp(min=0.0)
    alpha = (a_ess - beta * a_var).clamp(0.0, 1.0) * a_mis
    diag = torch.stack([mean_w, var_w, cv2, 1 / (1 + cv2), dbar, std_a, std_aw, dsigma, a_ess, a_mis, a_var, alpha,
                        (d > math.log(c)).double().mean(), -d.mean(), (old[valid].exp() - roll[valid].exp()).abs().mean()])
    wt = 1 + alpha * ((old - roll).clamp(max=math.log(c)).exp() - 1)
    rho = (logp - old).exp()
    ar = a32[resp]
    lo, hi = 1.0 - p.clip_eps, 1.0 + p.clip_eps
    active = torch.where(ar >= 0, rho <= hi, rho >= lo)
    obj = wt * torch.where(active, rho * ar, rho.clamp(lo, hi) * ar)
    dobj = torch.where(active, wt * ar * rho, torch.zeros_like(wt))
    if logp_ref is not None:
        q = logp_ref - logp
        obj = obj - p.beta_kl * (q.exp() - q - 1)
        dobj = dobj - p.beta_kl * (1 - q.exp())
    scale = torch.where(count > 0, 1.0 / (b * count), torch.zeros_like(count))[resp]
    zero = torch.zeros_like(wt)
    loss = -torch.where(valid, scale * obj, zero).sum().reshape(1)
    g = torch.where(valid, scale * dobj, zero) * p.inv_temperature
    return dict(adv=adv, count=None, diag=diag, loss=loss, wtilde=torch.where(valid, wt, zero), g=g)


def exact(case, seed):
    s = prepare(case, seed)
    n, v, kind, p = case["rows"], case["vocab"], case["kind"], s["params"]
    t = p.inv_temperature
    old = None if s["logp_old"] is None else s["logp_old"].double()
    ref = None if s["logp_ref"] is None else s["logp_ref"].double()
    if kind == "scalars":
        return exact_scalars(s, s["logp"].double(), old, ref)
    valid = torch.ones(n, dtype=torch.bool, device="cuda") if s["valid"] is None else s["valid"].bool()
    y = s["tokens"].long().clamp(min=0).unsqueeze(1)
    step = max(1, int(1.5e8) // v)
    if kind == "fp8_codes":
        codes = torch.empty(n, v, dtype=torch.uint8, device="cuda")
        scale = torch.empty(n, dtype=torch.float64, device="cuda")
        z8 = torch.empty(n, v, dtype=torch.float64, device="cuda")
        for r0 in range(0, n, step):
            z = s["logits"][r0:r0 + step].float()
            sc = z.abs().amax(dim=1) / torch.full((z.shape[0],), E4M3_MAX, device="cuda")
            sc = torch.where(sc > 0, sc, torch.ones_like(sc))
            code = (z / sc.unsqueeze(1)).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn)
            codes[r0:r0 + step] = code.view(torch.uint8)
            scale[r0:r0 + step] = sc.double()
            z8[r0:r0 + step] = code.double() * sc.double().unsqueeze(1)
        return dict(codes=codes, scale=scale, z=z8)

    def logits64(r0, r1):
        if kind in ("head_logprob", "head_step"):
            return s["hidden"][r0:r1].double() @ weight64.t() * t
        if kind == "fp8_logprob":
            return round_trip(s["logits"][r0:r1])
        return s["logits"][r0:r1].double() * t

    def round_trip(x):
        z = x.float()
        sc = z.abs().amax(dim=1, keepdim=True) / torch.full((z.shape[0], 1), E4M3_MAX, device="cuda")
        sc = torch.where(sc > 0, sc, torch.ones_like(sc))
        return (z / sc).clamp(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn).double() * sc.double()

    if kind in ("head_logprob", "head_step"):
        weight64 = s["weight"].double()
    lse, logp = torch.zeros(n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    for r0 in range(0, n, step):
        z = logits64(r0, min(n, r0 + step))
        lse[r0:r0 + step] = torch.logsumexp(z, dim=1)
        # log-prob of the token through the other tokens' share, which does not cancel where the token is near certain
        zy = z.gather(1, y[r0:r0 + step]).squeeze(1)
        z.scatter_(1, y[r0:r0 + step], -math.inf)
        logp[r0:r0 + step] = -torch.log1p((torch.logsumexp(z, dim=1) - zy).exp())
        del z
    lse[~valid] = 0.0
    logp[~valid] = 0.0
    if kind == "fp8_logprob":
        return logp
    if kind == "head_logprob":
        return dict(logp=logp, lse=lse)
    out = exact_scalars(s, logp, old, ref)
    out.update(logp=logp, lse=lse)
    g = out["g"]

    def direction(r0, r1, z):
        z.sub_(lse[r0:r1].unsqueeze(1)).exp_()
        z.scatter_(1, y[r0:r1], torch.expm1(logp[r0:r1]).unsqueeze(1))
        return z

    if kind == "head_step":
        out["dhidden"] = torch.zeros(n, case["d_model"], dtype=torch.float64, device="cuda")
        out["dweight"] = torch.zeros(v, case["d_model"], dtype=torch.float64, device="cuda")
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            ds = direction(r0, r1, logits64(r0, r1)).mul_(g[r0:r1].unsqueeze(1))
            out["dhidden"][r0:r1] = ds @ weight64
            out["dweight"] += ds.t().contiguous() @ s["hidden"][r0:r1].double()
            del ds
        return out
    dz = torch.zeros(n, v, dtype=torch.float64, device="cuda")
    for r0 in range(0, n, step):
        r1 = min(n, r0 + step)
        z = direction(r0, r1, logits64(r0, r1))
        dz[r0:r1] = z.mul_((g if kind == "step" else valid.double())[r0:r1].unsqueeze(1))
        del z
    if kind == "step":
        out["dlogits"] = dz
        del out["g"]
    else:
        out["sgrad"] = dz
    return out
