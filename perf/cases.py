"""Timed cases of the library: what a GRPO trainer calls, over the sizes it calls them with.

A case is one pass through the public entry points on synthetic inputs that already sit in
GPU memory.  ``path`` says which part of a training step it is:

  rewards       between rollouts and the step: length-penalised rewards, online filter, group
                advantages (per rollout and per token) and the packed layout; a few thousand
                values, so launches and their latency
  loss          one optimiser micro-batch on logits: advantages, then objective and gradient
  aux           the same on a packed batch with the KL and entropy terms and sample-level weights
  logprobs      the pass over the logits that recomputes the old policy's log-probs
  head_logprobs the same from hidden states and the language-model head's weights
  head_loss     objective, dL/dH and dL/dW from hidden states and weights
  head_aux      head_loss with the KL and entropy terms and sample-level weights

Vocabularies, dtypes, option values and distributions are those of the package's own workloads,
tests and benchmark: padded responses with the tail masked, 16 responses per prompt, binary
rewards, logits of standard deviation 3 with the sampled token raised by 8, old log-probs a
little off the new ones (a few far off, which populates every clip).
"""
import math

import torch

import paper_2505_07291_amd as grpo

EPS_LOW, EPS_HIGH, DELTA = 0.2, 0.2, 4.0
KL_COEF, ENT_COEF, ALPHA = 0.001, 1e-4, 3e-4
DEV = "cuda:0"
CHUNK = 1 << 28  # logits made or checked at a time


def listed():
    return [
        # the shaping of one small rollout step: 4 prompts of 16 responses, a few thousand tokens
        dict(name="rewards", path="rewards", groups=4, group_size=16, tokens=16384),
        # the smallest step in the package's workloads: launches and latency
        dict(name="loss_tiny", path="loss", rows=512, seq=64, vocab=1024, dtype="f32", temperature=1.0),
        # one short response as a micro-batch of its own: little more than a row for each compute unit
        dict(name="loss_micro", path="loss", rows=300, seq=300, vocab=152064, dtype="bf16", temperature=0.7),
        # the benchmark's batch: 64 responses of at most 256 tokens, a third of the rows masked
        dict(name="loss_short", path="loss", rows=16384, seq=256, vocab=152064, dtype="bf16", temperature=1.0),
        # a tokenizer whose vocabulary is used as it is, not padded: fp32 logits ...
        dict(name="loss_ragged_f32", path="loss", rows=4096, seq=256, vocab=50257, dtype="f32", temperature=1.0),
        # ... and bf16 logits of a large one, cut out of padded rows
        dict(name="loss_ragged_wide", path="loss", rows=4096, seq=512, vocab=152069, dtype="bf16", temperature=1.0),
        # a trainer that upcasts its logits before the loss
        dict(name="loss_f32", path="loss", rows=2048, seq=512, vocab=152064, dtype="f32", temperature=0.7),
        # a packed batch with all three terms, weighted per sample
        dict(name="aux_packed", path="aux", rows=8192, seq=512, vocab=128256, dtype="bf16", temperature=1.0),
        # old log-probs at the start of an optimiser step
        dict(name="logprobs_short", path="logprobs", rows=16384, seq=256, vocab=152064, dtype="bf16", temperature=1.0),
        # the same without logits in memory, for one long response
        dict(name="head_logprobs", path="head_logprobs", rows=2048, seq=1024, vocab=152064, d_model=5120, temperature=1.0),
        # a training micro-batch through the head of a 32B-sized model
        dict(name="head_loss", path="head_loss", rows=4096, seq=512, vocab=152064, d_model=5120, temperature=1.0),
        # a small model's micro-batch with all three terms
        dict(name="head_aux_small", path="head_aux", rows=1024, seq=128, vocab=50304, d_model=768, temperature=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, every size from a logarithmic spread."""
    path = rng.choice(["rewards", "loss", "loss", "loss", "aux", "logprobs", "head_logprobs", "head_loss", "head_aux"])
    if path == "rewards":
        return dict(path=path, groups=_log_int(rng, 2, 1024), group_size=rng.choice([2, 4, 8, 16, 32]),
                    tokens=_log_int(rng, 256, 1 << 18))
    case = dict(path=path, temperature=rng.choice([0.7, 1.0, 1.0]))
    if path.startswith("head"):
        case.update(vocab=_log_int(rng, 1000, 152064), d_model=64 * _log_int(rng, 4, 80))
        # at most the flops of the largest listed case
        case["rows"] = min(_log_int(rng, 64, 8192), 4096 * 152064 * 5120 // (case["vocab"] * case["d_model"]))
    else:
        case.update(vocab=_log_int(rng, 1000, 300000), dtype=rng.choice(["bf16", "bf16", "f32"]))
        if rng.random() < 0.6:  # most trainers pad the vocabulary
            case["vocab"] -= case["vocab"] % 64
        case["rows"] = min(_log_int(rng, 32, 32768), 16384 * 152064 * 2 // (case["vocab"] * _bytes(case)))
    case["seq"] = min(case["rows"], _log_int(rng, 16, 1024))
    return case


def _bytes(case):
    return 4 if case.get("dtype") == "f32" else 2


def _gen(seed, device="cpu"):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _rows(case, seed):
    """Everything per token or rollout: the responses lie one after the other, `seq` rows each (the
    last one takes what is left); the tail of each is padding.  Responses come in groups of 16."""
    g = _gen(seed)
    n, seq, group = case["rows"], case["seq"], 16
    n_resp = (n + seq - 1) // seq
    n_roll = (n_resp + group - 1) // group * group  # the other responses of a group may lie in other micro-batches
    rollout = torch.div(torch.arange(n), seq, rounding_mode="floor").to(torch.int32)
    length = torch.randint(max(1, seq // 4), seq + 1, (n_resp,), generator=g)
    mask = (torch.arange(n) % seq < length[rollout.long()]).to(torch.uint8)
    rewards = (torch.rand(n_roll, generator=g) < 0.3).float()
    rewards[::group] = 1.0  # one solved and one failed response at least: the group has a signal
    rewards[1::group] = 0.0
    tokens = torch.randint(0, case["vocab"], (n,), generator=g)
    noise = torch.randn(n, generator=g, dtype=torch.float64) * 0.1
    far = torch.rand(n, generator=g) < 0.02  # tokens of a response from an older policy
    noise[far] *= 20.0
    for kink in (math.log(1 - EPS_LOW), math.log(1 + EPS_HIGH), math.log(DELTA)):
        near = (-noise - kink).abs() < 1e-3  # which side of a clip such a token is on is rounding
        noise[near] -= 3e-3
    ref_noise = torch.randn(n, generator=g, dtype=torch.float64) * 0.05
    cu = torch.cat([torch.arange(n_resp) * seq, torch.tensor([n])])
    to = lambda t: t.to(DEV)  # noqa: E731
    return dict(n=n, n_resp=n_resp, group=group, rollout=to(rollout), mask=to(mask), rewards=to(rewards), tokens=to(tokens),
                noise=to(noise), ref_noise=to(ref_noise), cu=to(cu))


def _old_logprobs(s, case, lp):
    s["old"] = (lp.double() + s.pop("noise")).float()
    s["ref"] = (lp.double() + s.pop("ref_noise")).float()


def _logits(s, case, seed):
    n, v, dt = s["n"], case["vocab"], torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    per16 = 16 // _bytes(case)
    pitch = (v + per16 - 1) // per16 * per16  # rows start on 16-byte boundaries
    g = _gen(seed + 1, DEV)
    s["logits"] = torch.zeros((n, pitch), dtype=dt, device=DEV)[:, :v]
    lp = torch.empty(n, dtype=torch.float32, device=DEV)
    step = max(1, CHUNK // v)
    for a in range(0, n, step):
        y = s["tokens"][a:a + step, None]
        z = torch.randn((len(y), v), generator=g, device=DEV).mul_(3.0)
        z.scatter_add_(1, y, torch.full_like(y, 8.0, dtype=torch.float32))
        s["logits"][a:a + step] = z.to(dt)
        z = s["logits"][a:a + step].float().div_(case["temperature"])
        lp[a:a + step] = z.gather(1, y)[:, 0] - torch.logsumexp(z, 1)
    _old_logprobs(s, case, lp)


def _head(s, case, seed):
    n, v, d = s["n"], case["vocab"], case["d_model"]
    g = _gen(seed + 1, DEV)
    s["weight"] = torch.randn((v, d), generator=g, device=DEV).mul_(3.0 / math.sqrt(d)).to(torch.bfloat16)
    wy = s["weight"][s["tokens"]].float()
    h = torch.randn((n, d), generator=g, device=DEV)
    s["hidden"] = (h + 8.0 * wy / (wy * wy).sum(1, keepdim=True)).to(torch.bfloat16)
    w = s["weight"].float()
    lp = torch.empty(n, dtype=torch.float32, device=DEV)
    for a in range(0, n, 2048):
        z = (s["hidden"][a:a + 2048].float() @ w.t()).div_(case["temperature"])
        lp[a:a + 2048] = z.gather(1, s["tokens"][a:a + 2048, None])[:, 0] - torch.logsumexp(z, 1)
    _old_logprobs(s, case, lp)


def prepare(case, seed):
    path = case["path"]
    if path == "rewards":
        g = _gen(seed)
        n = case["groups"] * case["group_size"]
        t = case["tokens"]
        lengths = torch.randint(1, max(2, t // n + 1), (n,), generator=g)
        solved = (torch.rand(n, generator=g) < 0.5).float()
        every = torch.rand(case["groups"], generator=g) < 0.25  # prompts that all or no response solves
        solved = torch.where(every.repeat_interleave(case["group_size"]), 1.0, solved)
        cu = torch.cat([torch.zeros(1, dtype=torch.int64), lengths.cumsum(0)]).clamp(max=t)
        # a quarter of the prompts ask for no length: their responses' penalties are zero
        target = torch.where(every.repeat_interleave(case["group_size"]), lengths, torch.randint(1, 4096, (n,), generator=g))
        return dict(case=case, task=solved.to(DEV), lengths=lengths.int().to(DEV), target=target.int().to(DEV), cu=cu.to(DEV),
                    tokens=t)
    s = _rows(case, seed)
    s["case"] = case
    n = s["n"]
    if path.startswith("head"):
        _head(s, case, seed)
        v, d = case["vocab"], case["d_model"]
        train = path != "head_logprobs"
        s["workspace"] = torch.empty(grpo.grpo_lmhead_workspace_bytes(n, v, d, train), dtype=torch.uint8, device=DEV)
        if train:
            s["grad_hidden"] = torch.empty((n, d), dtype=torch.bfloat16, device=DEV)
            s["grad_weight"] = torch.empty((v, d), dtype=torch.float32, device=DEV)
    else:
        _logits(s, case, seed)
        if path != "logprobs":
            s["workspace"] = torch.empty(grpo.grpo_workspace_bytes(n), dtype=torch.uint8, device=DEV)
            s["grad"] = torch.empty_strided(s["logits"].shape, s["logits"].stride(), dtype=s["logits"].dtype, device=DEV)
    return s


def run(s):
    case = s["case"]
    path, temp = case["path"], case.get("temperature")
    if path == "rewards":
        rewards = grpo.grpo_total_rewards(s["task"], s["lengths"], s["target"], ALPHA)
        keep, kept, n_kept, rollout_keep = grpo.grpo_filter_groups(rewards, group_size=case["group_size"])
        weights, rollout = grpo.grpo_packed_layout(s["cu"], s["tokens"], sample_level=True)
        adv, adv_tok = grpo.grpo_group_advantages(rewards, group_size=case["group_size"], rollout_of_token=rollout)
        return dict(rewards=rewards, keep=keep, kept=kept, n_kept=n_kept, rollout_keep=rollout_keep, weights=weights,
                    rollout=rollout, adv=adv, adv_tok=adv_tok)
    if path == "logprobs":
        return grpo.grpo_logprobs_fwd(s["logits"], s["tokens"], s["mask"], temp)
    if path == "head_logprobs":
        return grpo.grpo_lmhead_logprobs_fwd(s["hidden"], s["weight"], s["tokens"], s["mask"], temp, workspace=s["workspace"])
    rollout = s["rollout"]
    if path in ("aux", "head_aux"):
        weights, rollout = grpo.grpo_packed_layout(s["cu"], s["n"], sample_level=True)
    _, adv = grpo.grpo_group_advantages(s["rewards"], group_size=s["group"], rollout_of_token=rollout)
    if path == "loss":
        loss, lp, counts, grad = grpo.grpo_loss_fwd_bwd(
            s["logits"], s["tokens"], s["old"], adv, s["mask"], EPS_LOW, EPS_HIGH, DELTA, temp, grad_logits=s["grad"],
            workspace=s["workspace"])
        return dict(loss=loss, logprobs=lp, counts=counts, grad=grad)
    if path == "aux":
        loss, lp, ent, counts, grad = grpo.grpo_loss_aux_fwd_bwd(
            s["logits"], s["tokens"], s["old"], s["ref"], adv, s["mask"], EPS_LOW, EPS_HIGH, DELTA, temp, KL_COEF, ENT_COEF,
            denom=float(s["n_resp"]), token_weights=weights, grad_logits=s["grad"], workspace=s["workspace"])
        return dict(loss=loss, logprobs=lp, entropy=ent, counts=counts, grad=grad)
    if path == "head_loss":
        loss, lp, counts, gh, gw = grpo.grpo_lmhead_loss_fwd_bwd(
            s["hidden"], s["weight"], s["tokens"], s["old"], adv, s["mask"], EPS_LOW, EPS_HIGH, DELTA, temp,
            grad_hidden=s["grad_hidden"], grad_weight=s["grad_weight"], workspace=s["workspace"])
        return dict(loss=loss, logprobs=lp, counts=counts, grad_hidden=gh, grad_weight=gw)
    loss, lp, ent, counts, gh, gw = grpo.grpo_lmhead_loss_aux_fwd_bwd(
        s["hidden"], s["weight"], s["tokens"], s["old"], s["ref"], adv, s["mask"], EPS_LOW, EPS_HIGH, DELTA, temp, KL_COEF,
        ENT_COEF, denom=float(s["n_resp"]), token_weights=weights, grad_hidden=s["grad_hidden"], grad_weight=s["grad_weight"],
        workspace=s["workspace"])
    return dict(loss=loss, logprobs=lp, entropy=ent, counts=counts, grad_hidden=gh, grad_weight=gw)


def work(case):
    """Rows that take part: five eighths of them on average (the padded tail of a response is uniform)."""
    path = case["path"]
    if path == "rewards":
        n = case["groups"] * case["group_size"]
        return dict(bytes=n * 40 + case["groups"] * 5 + case["tokens"] * 12, flops=n * 8)
    n, v, live = case["rows"], case["vocab"], case["rows"] * 0.625
    if path.startswith("head"):
        d = case["d_model"]
        products = 1 if path == "head_logprobs" else 3
        wide = v * d * 2 + n * 20 + live * d * 2
        return dict(bytes=wide if products == 1 else wide + v * d * 4 + n * d * 2, flops=2.0 * products * live * v * d)
    row = v * _bytes(case)
    return dict(bytes=live * row + n * 13 if path == "logprobs" else live * row + n * row + n * 25, flops=live * v * (5 if path == "logprobs" else 9))


def tolerance(case):
    """What another order of the same arithmetic may differ by.  Against fp64 the log-probs measure 4e-8 to 4e-7,
    fp32 gradients 3e-7 to 7e-7 (exponents of up to 2^5 carry 2^-19 into single probabilities) and bf16 ones
    1.2e-3 to 1.8e-3, which is their rounding; the head's gradients 1.4e-3 to 2.5e-3, where G is rounded to
    bf16 in front of the two products."""
    path = case["path"]
    if path == "rewards":
        return {"rel": 1e-6}
    if path in ("logprobs", "head_logprobs"):
        return {"rel": 1e-5}
    if path.startswith("head") or case["dtype"] == "bf16":
        return {"rel": 4e-3, "max": 0.1}
    return {"rel": 1e-5, "max": 1e-3}


def _objective(lp, old, adv, mask, weight, denom):
    """J and dJ/dl in fp64 (a ratio on a boundary counts as not clipped)."""
    r = torch.exp(lp - old)
    s1, s2 = r.clamp(max=DELTA) * adv, r.clamp(1 - EPS_LOW, 1 + EPS_HIGH) * adv
    opened = torch.where(s1 <= s2, r <= DELTA, (r >= 1 - EPS_LOW) & (r <= 1 + EPS_HIGH))
    on = mask != 0
    count = lambda c: (c & on).sum()  # noqa: E731
    counts = torch.stack([on.sum(), count((adv > 0) & (r > 1 + EPS_HIGH)), count((adv < 0) & (r < 1 - EPS_LOW)),
                          count((adv < 0) & (r > DELTA)), count((r < 1 - EPS_LOW) | (r > 1 + EPS_HIGH))])
    w = weight * on
    return torch.minimum(s1, s2), torch.where(opened, adv * r, 0.0), w / denom, counts


def _advantages(s):
    r = s["rewards"].double().view(-1, s["group"])
    a = (r - r.mean(1, keepdim=True)) / (r.std(1, keepdim=True, correction=0) + 1e-6)
    return a.flatten()[s["rollout"].long()]


def exact(case, seed):
    """The same in fp64 with plain torch."""
    s = prepare(case, seed)
    path, temp = case["path"], case.get("temperature")
    if path == "rewards":
        rewards = s["task"].double() - ALPHA * (s["target"].double() - s["lengths"].double()).abs()
        r = rewards.view(case["groups"], -1)
        # the advantages of rewards that fp32 has rounded, as the trainer stores them
        r32 = r.float().double()
        adv = (r32 - r32.mean(1, keepdim=True)) / (r32.std(1, keepdim=True, correction=0) + 1e-6)
        adv = adv.flatten()
        t = torch.arange(s["tokens"], device=DEV)
        rollout = torch.searchsorted(s["cu"], t, right=True) - 1
        own = rollout < s["cu"].numel() - 1
        at = rollout.clamp(max=s["cu"].numel() - 2)
        length = (s["cu"][1:] - s["cu"][:-1]).double()
        return dict(rewards=rewards, keep=None, kept=None, n_kept=None, rollout_keep=None,
                    weights=torch.where(own, 1.0 / length[at], 0.0), rollout=None, adv=adv, adv_tok=torch.where(own, adv[at], math.nan))
    n, v, tokens, mask = s["n"], case["vocab"], s["tokens"], s["mask"]
    head, aux = path.startswith("head"), path in ("aux", "head_aux")
    adv = _advantages(s)
    on = mask != 0
    length = torch.bincount(s["rollout"].long(), minlength=s["n_resp"]).double()
    weight = 1.0 / length[s["rollout"].long()] if aux else torch.ones(n, dtype=torch.float64, device=DEV)
    denom = float(s["n_resp"]) if aux else float(on.sum())
    lp, ent, kl = (torch.zeros(n, dtype=torch.float64, device=DEV) for _ in range(3))
    train = path not in ("logprobs", "head_logprobs")
    jj, wd = torch.zeros(n, dtype=torch.float64, device=DEV), torch.zeros(n, dtype=torch.float64, device=DEV)
    counts = torch.zeros(5, dtype=torch.int64, device=DEV)
    w64 = s["weight"].double() if head else None
    if head and train:
        gh = torch.zeros((n, case["d_model"]), dtype=torch.float64, device=DEV)
        gw = torch.zeros((v, case["d_model"]), dtype=torch.float64, device=DEV)
    elif train:
        gl = torch.empty((n, v), dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // v)
    for a in range(0, n, step):
        b = slice(a, min(n, a + step))
        y = tokens[b, None]
        z = (s["hidden"][b].double() @ w64.t() if head else s["logits"][b].double()) / temp
        z -= torch.logsumexp(z, 1, keepdim=True)
        lp[b] = z.gather(1, y)[:, 0]
        if not train:
            continue
        jj[b], dj, wd[b], c = _objective(lp[b], s["old"][b].double(), adv[b], mask[b], weight[b], denom)
        counts += c
        cy = -dj * wd[b]
        p = z.exp()
        if aux:
            d = s["ref"][b].double() - lp[b]
            kl[b] = torch.exp(d) - d - 1
            ent[b] = -(p * z).sum(1)
            cy += KL_COEF * (1 - torch.exp(d)) * wd[b]
            z += ent[b, None]
            z *= (ENT_COEF * wd[b])[:, None]
            z -= cy[:, None]
        else:
            z = (-cy)[:, None].expand_as(p)
        p *= z
        p.scatter_add_(1, y, cy[:, None])
        p /= temp
        if head:
            gh[b] = p @ w64
            gw += p.t() @ s["hidden"][b].double()
        else:
            gl[b] = p
        del p, z
    lp, ent = lp * on, ent * on
    if not train:
        return lp
    policy, mean_kl, mean_ent = -(jj * wd).sum(), (kl * wd).sum(), (ent * wd).sum()
    loss = torch.stack([policy + KL_COEF * mean_kl - ENT_COEF * mean_ent, policy, mean_kl, mean_ent]) if aux else policy[None]
    out = dict(loss=loss, logprobs=lp, counts=None)
    if aux:
        out["entropy"] = ent
    if head:
        return dict(out, grad_hidden=gh, grad_weight=gw)
    return dict(out, grad=gl)
