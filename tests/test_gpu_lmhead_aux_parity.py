"""GPU parity of the fused language-model-head path with the auxiliary terms
(grpo_lmhead_loss_aux_fwd_bwd: policy term, sampled-token KL, entropy bonus, per-token
weights, on logits the library forms itself) against the fp64 oracle.

Tolerances: scalars and per-token outputs as for the logits path with the auxiliary terms
(log-probs 2e-4 abs, per-token entropy 2e-4 abs, total / policy 1e-4 rel, mean KL 1e-4 rel
+ 1e-9, mean entropy 1e-4 rel + 2e-7, counters exact); dL/dH and dL/dW as for the plain
head path: G is rounded to bf16 (u = 2^-8) before the two fp32-accumulating products and
dL/dH is rounded to bf16 on output, so element by element
    |d dH[t,k]| <= u sum_v |G[t,v]| |W[v,k]| + u |dH[t,k]|,   |d dW[v,k]| <= u sum_t |G[t,v]| |H[t,k]|
with 5 % slack, plus what the logits path's gradient bound adds for the two new terms, carried
through the products: the KL part of a row's coefficient is known to two fp32 ulps of l
(floor_kl = |kl_coef grad_scale omega / (D T)| 2^-22 max(|l|, 1) on every |G[t,v]| of the row via
p_v, i.e. floor_kl * sum_v p_v |W[v,k]| <= floor_kl max|W|), and the entropy part to
|ent_coef grad_scale omega / (D T)| p_max max(H, 1) 2^-20; and the error must look like
rounding noise (Frobenius norm below 0.6 u of the norm of the bounds).
"""
import numpy as np
import pytest
import torch

import paper_2505_07291_amd as grpo
from paper_2505_07291_amd import workloads as wl
from oracle import grpo_oracle as orc
from test_gpu_lmhead_parity import DEV, TOL_LOGP, TOL_LOSS_REL, U, bits, f32, say, wide

pytestmark = pytest.mark.gpu


def run_aux_case(cfg, d_model, kl_coef, ent_coef, *, denom=0.0, grad_scale=1.0, weighted=False, label="",
                 batch=None):
    if batch is None:
        batch = wl.make_lmhead_batch(cfg, d_model, device=DEV)
    N, V = batch["n_tokens"], batch["vocab"]
    T = f32(cfg.temperature)
    kw = dict(eps_low=f32(cfg.eps_low), eps_high=f32(cfg.eps_high), delta=f32(cfg.delta))
    hb, wb = bits(batch["hidden"]), bits(batch["weight"])
    tokens_np, mask_np = batch["tokens"].cpu().numpy(), batch["mask"].cpu().numpy()
    adv = orc.group_advantages(batch["rewards"].cpu().numpy(), group_size=batch["group_size"])
    adv_tok = orc.broadcast_advantages(adv, batch["rollout_of_token"].cpu().numpy()).astype(np.float32)
    lp_orc = orc.logprobs(orc.lmhead_logits(hb, wb), tokens_np, mask_np, temperature=T)
    old = wl.make_old_logprobs(cfg, lp_orc)
    g = torch.Generator().manual_seed(1900 + cfg.index)
    ref = (torch.as_tensor(lp_orc) + torch.randn(N, generator=g, dtype=torch.float64) * 0.1).float()
    tw = None
    if weighted:
        tw = (torch.rand(N, generator=g) * 1.3 + 0.2).float()
        tw[::7] = 0.0                                   # zero weight: the row drops out like a masked one
    tw_np = None if tw is None else tw.numpy()
    want = orc.lmhead_aux_loss_fwd_bwd(hb, wb, tokens_np, old.numpy(), ref.numpy(), adv_tok, mask_np,
                                       token_weights=tw_np, temperature=T, kl_coef=f32(kl_coef),
                                       ent_coef=f32(ent_coef), denom=denom, grad_scale=f32(grad_scale), **kw)
    say("[gpu] %s grpo_lmhead_loss_aux_fwd_bwd N=%d V=%d d=%d kl=%g ent=%g" % (label, N, V, d_model, kl_coef, ent_coef))
    loss, lp, ent, counts, dH, dW = grpo.grpo_lmhead_loss_aux_fwd_bwd(
        batch["hidden"], batch["weight"], batch["tokens"], old.to(DEV), ref.to(DEV),
        torch.as_tensor(adv_tok, device=DEV), batch["mask"], temperature=T, kl_coef=kl_coef,
        entropy_coef=ent_coef, denom=denom, grad_scale=grad_scale,
        token_weights=None if tw is None else tw.to(DEV), **kw)
    torch.cuda.synchronize()
    got = loss.cpu().numpy().astype(np.float64)
    e_lp = np.abs(lp.cpu().numpy() - want["logprobs"]).max()
    e_h = np.abs(ent.cpu().numpy() - want["entropies"]).max()
    say("      |dl|=%.1e |dH_t|=%.1e total %.8g vs %.8g kl %.5g H %.6g counts %s" %
        (e_lp, e_h, got[0], want["total"], got[2], got[3], counts.tolist()))
    assert e_lp <= TOL_LOGP and e_h <= 2e-4
    assert counts.cpu().numpy().tolist() == want["counts"].tolist()
    assert abs(got[0] - want["total"]) <= TOL_LOSS_REL * abs(want["total"]) + 1e-7
    assert abs(got[1] - want["policy"]) <= TOL_LOSS_REL * abs(want["policy"]) + 1e-7
    assert abs(got[2] - want["kl"]) <= 1e-4 * want["kl"] + 1e-9
    assert abs(got[3] - want["entropy"]) <= 1e-4 * want["entropy"] + 2e-7
    # gradients
    G = want["grad"]
    H64, W64 = wide(hb), wide(wb)
    M = int(want["counts"][0])
    D = denom if denom > 0 else float(max(M, 1))
    wrow = np.ones(N) if tw_np is None else np.abs(tw_np.astype(np.float64))
    scale = wrow * abs(f32(grad_scale)) / (D * T)
    z = want["logits"]
    pmax = np.exp(z.max(axis=1) / T - z[np.arange(N), tokens_np] / T + want["logprobs"])
    floor_row = scale * (abs(f32(kl_coef)) * 2.0 ** -22 * np.maximum(np.abs(want["logprobs"]), 1.0) +
                         abs(f32(ent_coef)) * pmax * np.maximum(want["entropies"], 1.0) * 2.0 ** -20)
    floor_row = np.where((mask_np == 1) & (wrow > 0), floor_row, 0.0)
    bH = U * (np.abs(G) @ np.abs(W64) + np.abs(want["grad_hidden"])) + floor_row[:, None] * np.abs(W64).max()
    bW = U * (np.abs(G).T @ np.abs(H64)) + (floor_row[:, None] * np.abs(H64)).sum(axis=0)[None, :]
    eH = np.abs(dH.cpu().double().numpy() - want["grad_hidden"])
    eW = np.abs(dW.cpu().double().numpy() - want["grad_weight"])
    say("      dH err max %.3e (max %.3e)  dW err max %.3e (max %.3e)" %
        (eH.max(), np.abs(want["grad_hidden"]).max(), eW.max(), np.abs(want["grad_weight"]).max()))
    assert np.all(eH <= 1.05 * bH + 1e-30), "dH off by %g of its bound" % (eH / (bH + 1e-300)).max()
    assert np.all(eW <= 1.05 * bW + 1e-30), "dW off by %g of its bound" % (eW / (bW + 1e-300)).max()
    assert np.linalg.norm(eH) <= 0.6 * np.linalg.norm(bH) and np.linalg.norm(eW) <= 0.6 * np.linalg.norm(bW)
    nograd = (want["coeff"] == 0) & (want["ent_coeff"] == 0)
    assert not dH.cpu().float().numpy()[nograd].any()
    return batch, want


SHAPES = [
    ("qwen_short", 2, 4, 64, 1000, 128),
    ("qwen_medium", 2, 4, 100, 2600, 192),
    ("long_reasoning", 4, 4, 40, 1300, 320),
    ("numerics_stress", 2, 4, 64, 900, 128),
]


@pytest.mark.parametrize("name,P,G,L,V,D", SHAPES)
@pytest.mark.parametrize("coefs", [(0.001, 1e-4), (0.05, 0.02)], ids=["paper_coefs", "large_coefs"])
def test_reduced_configs_every_element(name, P, G, L, V, D, coefs):
    cfg = wl.CONFIGS[name].scaled(n_prompts=P, seq_len=L, vocab=V, group_size=G)
    if cfg.logits not in ("normal", "normal_boost"):
        cfg = wl.replace(cfg, logits="normal", logit_std=3.0)
    run_aux_case(cfg, D, coefs[0], coefs[1], label="%s %dx%dx%d" % (name, P * G * L, V, D))


def test_near_one_hot_rows():
    """Rows whose hidden state points along one weight row, so that one logit stands 40 to 50
    above the rest: on the sampled token (p_y within 1e-15 of 1: the ln(1 + x) form of l, an
    entropy of order 1e-14 and gradients that vanish) or on another token (l near -45)."""
    cfg = wl.CONFIGS["qwen_short"].scaled(n_prompts=2, seq_len=32, vocab=1100, group_size=4)
    d = 128
    batch = wl.make_lmhead_batch(cfg, d, device=DEV)
    N, V = batch["n_tokens"], batch["vocab"]
    W = batch["weight"].float()
    g = torch.Generator().manual_seed(4242)
    other = torch.randint(0, V, (N,), generator=g).to(DEV)
    target = torch.where(torch.arange(N, device=DEV) % 4 < 2, batch["tokens"], other)   # half on y, a quarter elsewhere
    wy = W[target]
    spike = 45.0 * wy / (wy * wy).sum(dim=1, keepdim=True)
    noise = torch.randn((N, d), generator=g).to(DEV) * 0.05
    spiked = (torch.arange(N, device=DEV) % 4 != 3)[:, None]
    batch["hidden"] = torch.where(spiked, spike + noise, batch["hidden"].float()).to(torch.bfloat16).contiguous()
    run_aux_case(cfg, d, 0.05, 0.02, label="near one-hot", batch=batch)


def test_token_weights_denominator_and_grad_scale():
    cfg = wl.CONFIGS["qwen_short"].scaled(n_prompts=2, seq_len=40, vocab=1500, group_size=4)
    run_aux_case(cfg, 128, 0.05, 0.02, denom=8.0, grad_scale=2.5, weighted=True, label="weights/denom/scale")


def test_zero_coefficients_match_the_plain_head_call_and_rows_without_gradient_stay_zero():
    cfg = wl.CONFIGS["numerics_stress"].scaled(n_prompts=2, seq_len=48, vocab=700, group_size=4)
    cfg = wl.replace(cfg, logits="normal", logit_std=3.0)
    b = wl.make_lmhead_batch(cfg, 128, device=DEV)
    lp0 = grpo.grpo_lmhead_logprobs_fwd(b["hidden"], b["weight"], b["tokens"], b["mask"])
    torch.cuda.synchronize()
    old = wl.make_old_logprobs(cfg, lp0).to(DEV)
    _, adv = grpo.grpo_group_advantages(b["rewards"], group_size=cfg.group_size, rollout_of_token=b["rollout_of_token"])
    kw = dict(eps_low=f32(cfg.eps_low), eps_high=f32(cfg.eps_high), delta=f32(cfg.delta))
    a = grpo.grpo_lmhead_loss_fwd_bwd(b["hidden"], b["weight"], b["tokens"], old, adv, b["mask"], **kw)
    c = grpo.grpo_lmhead_loss_aux_fwd_bwd(b["hidden"], b["weight"], b["tokens"], old, None, adv, b["mask"], **kw)
    torch.cuda.synchronize()
    assert torch.equal(a[2], c[3])                                   # counters
    assert abs(float(a[0]) - float(c[0][0])) <= 1e-4 * abs(float(a[0])) and float(c[0][2]) == 0.0
    assert float((a[1] - c[1]).abs().max()) <= TOL_LOGP
    dHa, dHc = a[3].float(), c[4].float()
    assert bool(((dHa == 0).all(dim=1) == (dHc == 0).all(dim=1)).all())   # the same rows have no gradient
    tol = 2.0 * U * dHa.abs().amax() + 1e-12
    assert float((dHa - dHc).abs().max()) <= tol
    assert float((a[4] - c[5]).abs().max()) <= 2.0 * U * float(a[4].abs().max()) + 1e-12
    # run to run: identical bits
    c2 = grpo.grpo_lmhead_loss_aux_fwd_bwd(b["hidden"], b["weight"], b["tokens"], old, None, adv, b["mask"], **kw)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(c, c2) if x is not None)


def test_full_size_qwen_short():
    """The benchmark's headline batch (16384 tokens, vocabulary 152064) with a 5120-wide head and the
    coefficients of section 4.1.  The oracle forms the fp64 logits of every unmasked row (its library
    products, pinned against its loops), so every input of the call and every expected value is the
    oracle's: log-probs and entropies of all rows, the four scalars and the counters; dL/dH element by
    element on 1024 sampled rows, dL/dW on 600 sampled vocabulary entries (every row with a gradient
    contributes to each), and the identities that tie the whole of dL/dW to dL/dH."""
    cfg = wl.CONFIGS["qwen_short"]
    d = 5120
    batch = wl.make_lmhead_batch(cfg, d, device=DEV)
    N, V = batch["n_tokens"], batch["vocab"]
    T = f32(cfg.temperature)
    kw = dict(eps_low=f32(cfg.eps_low), eps_high=f32(cfg.eps_high), delta=f32(cfg.delta))
    klc, enc = 0.001, 1e-4
    mask_np, tokens_np = batch["mask"].cpu().numpy(), batch["tokens"].cpu().numpy()
    unm = np.flatnonzero(mask_np != 0)
    M = len(unm)
    hb, wb = bits(batch["hidden"]), bits(batch["weight"])
    say("[gpu] full-size lmhead aux: oracle logits of the %d unmasked rows" % M)
    z = orc.lmhead_products("library")[0](hb[unm], wb)                  # [unmasked, V] fp64
    lp_orc, H_orc = np.zeros(N), np.zeros(N)
    lp_orc[unm] = orc.logprobs(z, tokens_np[unm], None, temperature=T)
    H_orc[unm] = orc.entropies(z, None, temperature=T)
    old = wl.make_old_logprobs(cfg, lp_orc)
    g = torch.Generator().manual_seed(1900 + cfg.index)
    ref = (torch.as_tensor(lp_orc) + torch.randn(N, generator=g, dtype=torch.float64) * 0.1).float()
    adv = orc.group_advantages(batch["rewards"].cpu().numpy(), group_size=batch["group_size"])
    adv_tok = orc.broadcast_advantages(adv, batch["rollout_of_token"].cpu().numpy()).astype(np.float32)
    want = orc.aux_objective_from_logprobs(lp_orc, H_orc, old.numpy(), ref.numpy(), adv_tok, mask_np,
                                           kl_coef=f32(klc), ent_coef=f32(enc), **kw)

    say("[gpu] full-size lmhead aux: grpo_lmhead_loss_aux_fwd_bwd N=%d V=%d d=%d" % (N, V, d))
    loss, lp, ent, counts, dH, dW = grpo.grpo_lmhead_loss_aux_fwd_bwd(
        batch["hidden"], batch["weight"], batch["tokens"], old.to(DEV), ref.to(DEV),
        torch.as_tensor(adv_tok, device=DEV), batch["mask"], temperature=T, kl_coef=klc, entropy_coef=enc, **kw)
    torch.cuda.synchronize()
    e_lp = np.abs(lp.cpu().numpy().astype(np.float64) - lp_orc).max()
    e_h = np.abs(ent.cpu().numpy().astype(np.float64) - H_orc).max()
    got = loss.cpu().numpy().astype(np.float64)
    say("[gpu] full-size lmhead aux: |dl| %.2e |dH_t| %.2e over all rows; total %.8g vs %.8g kl %.5g H %.6g counts %s" %
        (e_lp, e_h, got[0], want["total"], got[2], got[3], counts.tolist()))
    assert e_lp <= TOL_LOGP and e_h <= 2e-4
    assert counts.cpu().numpy().tolist() == want["counts"].tolist()
    assert abs(got[0] - want["total"]) <= TOL_LOSS_REL * abs(want["total"]) + 1e-7
    assert abs(got[1] - want["policy"]) <= TOL_LOSS_REL * abs(want["policy"]) + 1e-7
    assert abs(got[2] - want["kl"]) <= 1e-4 * want["kl"] + 1e-9
    assert abs(got[3] - want["entropy"]) <= 1e-4 * want["entropy"] + 2e-7

    # gradient with respect to the logits of every unmasked row, and the floors of run_aux_case per row
    coeff, ecoef = want["coeff"], want["ent_coeff"]
    pmax = np.exp(z.max(axis=1) / T - z[np.arange(M), tokens_np[unm]] / T + lp_orc[unm])
    G = orc.aux_grad_rows(z, tokens_np[unm], coeff[unm], ecoef[unm], temperature=T)
    del z
    floor_row = (klc * 2.0 ** -22 * np.maximum(np.abs(lp_orc[unm]), 1.0) +
                 enc * pmax * np.maximum(H_orc[unm], 1.0) * 2.0 ** -20) / (M * T)
    Wd, Hd = wide(wb), wide(hb[unm])
    rng = np.random.default_rng(23)
    pick = np.sort(rng.choice(M, 1024, replace=False))
    dH_o = G[pick] @ Wd
    bH = U * (np.abs(G[pick]) @ np.abs(Wd) + np.abs(dH_o)) + floor_row[pick, None] * np.abs(Wd).max()
    dH_np = dH.cpu().double().numpy()
    eH = np.abs(dH_np[unm[pick]] - dH_o)
    say("[gpu] full-size lmhead aux: dH err max %.3e (max|dH| %.3e) on %d rows" % (eH.max(), np.abs(dH_o).max(), len(pick)))
    assert np.all(eH <= 1.05 * bH + 1e-30), "dH off by %g of its bound" % (eH / (bH + 1e-300)).max()
    assert np.linalg.norm(eH) <= 0.6 * np.linalg.norm(bH)
    assert not dH_np[mask_np == 0].any()
    used = np.unique(tokens_np[unm])
    vs = np.unique(np.concatenate([rng.choice(used, 300, replace=False), rng.choice(V, 300, replace=False)]))
    Gs = np.ascontiguousarray(G[:, vs])
    dW_o = Gs.T @ Hd
    bW = U * (np.abs(Gs).T @ np.abs(Hd)) + (floor_row[:, None] * np.abs(Hd)).sum(axis=0)[None, :]
    eW = np.abs(dW.cpu().double().numpy()[vs] - dW_o)
    say("[gpu] full-size lmhead aux: dW err max %.3e (max|dW| %.3e) on %d vocabulary entries" %
        (eW.max(), np.abs(dW_o).max(), len(vs)))
    assert np.all(eW <= 1.05 * bW + 1e-30), "dW off by %g of its bound" % (eW / (bW + 1e-300)).max()
    assert np.linalg.norm(eW) <= 0.6 * np.linalg.norm(bW)
    del G, Gs
    inner_W = (dW.double() * batch["weight"].double()).sum().item()
    inner_H = (dH.double() * batch["hidden"].double()).sum().item()
    scale = (dW.double().abs() * batch["weight"].double().abs()).sum().item()
    say("[gpu] full-size lmhead aux: <dW,W> %.6e <dH,H> %.6e (scale %.3e)" % (inner_W, inner_H, scale))
    assert abs(inner_W - inner_H) <= U * scale
    col = dW.double().sum(dim=0).abs().max().item()
    assert col <= U * dW.double().abs().sum(dim=0).max().item()


@pytest.mark.parametrize("first,last", [(100, 101), (192, 256), (256, 320), (320, 321)])
def test_nan_in_the_weights_reaches_every_row(first, last):
    """A vocabulary entry whose weight row is NaN has a NaN logit in every row: log-probs, loss and gradients are
    NaN, also where a whole 64-column part of a tile, or all that a part has inside the matrix, is NaN (the last
    of 321 entries is alone in its part) and no number is left to be its maximum."""
    V, d, n = 321, 64, 70
    g = torch.Generator().manual_seed(first)
    w = (torch.randn((V, d), generator=g) * 0.3).to(torch.bfloat16)
    w[first:last] = float("nan")
    w, h = w.to(DEV), torch.randn((n, d), generator=g).to(torch.bfloat16).to(DEV)
    tok = torch.randint(0, 90, (n,), generator=g).to(DEV)
    old, adv = torch.full((n,), -6.0, device=DEV), torch.randn(n, generator=g).to(DEV)
    assert bool(torch.isnan(grpo.grpo_lmhead_logprobs_fwd(h, w, tok)).all())
    loss, lp, _, dH, _ = grpo.grpo_lmhead_loss_fwd_bwd(h, w, tok, old, adv)
    aux = grpo.grpo_lmhead_loss_aux_fwd_bwd(h, w, tok, old, old, adv, kl_coef=0.01, entropy_coef=0.01)
    torch.cuda.synchronize()
    assert bool(torch.isnan(lp).all()) and bool(torch.isnan(loss).all()) and bool(torch.isnan(dH.float()).all())
    assert bool(torch.isnan(aux[1]).all()) and bool(torch.isnan(aux[2]).all()) and bool(torch.isnan(aux[0]).all())
    assert bool(torch.isnan(aux[4].float()).all())


@pytest.mark.parametrize("adv,ref,sign", [(float("inf"), 0.0, 1), (float("-inf"), 0.0, -1), (1.0, float("inf"), 1),
                                          (float("nan"), 0.0, 0)])
def test_coefficients_that_are_no_finite_numbers(adv, ref, sign):
    """An infinite advantage or KL term makes dL/dz of its row infinite, with the sign that it has off the sampled token, and so
    dL/dW off that token's entry; one that is NaN makes it NaN."""
    n, v, d = 5, 700, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    h = torch.randn((n, d), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((v, d), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    tok = torch.randint(0, v, (n,), generator=g, device="cuda")
    lp = grpo.grpo_lmhead_logprobs_fwd(h, w, tok)
    a, r = torch.ones(n, device="cuda"), lp - 0.1
    a[2], r[2] = adv, lp[2] + ref
    out = grpo.grpo_lmhead_loss_aux_fwd_bwd(h, w, tok, lp + 0.05, r, a, None, kl_coef=0.01, entropy_coef=0.01)
    dH, dW = out[-2].float(), out[-1]
    assert bool(torch.isfinite(dH[[0, 1, 3, 4]]).all()) and not bool(torch.isfinite(dH[2]).any())
    off = torch.arange(v, device="cuda") != tok[2]
    if sign == 0:
        assert bool(torch.isnan(dW).all())
    else:
        assert bool((h[2] != 0).all())
        assert torch.equal(dW[off], (h[2].float() * sign * float("inf")).expand(int(off.sum()), d))
