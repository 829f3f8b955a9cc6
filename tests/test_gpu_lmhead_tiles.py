"""Sizes at which the head's products change how they divide their work: rows around 128 and 256 (whole, thin and
halved tiles, thin ones two to a place), vocabularies around the 64 columns of a wavefront's part and the 256 of a tile, one and two K steps,
contractions that are cut and that are not.  Against the fp64 oracle, element by element (run_case)."""
import pytest
import torch

import paper_2505_07291_amd as grpo
import paper_2505_07291_amd.workloads as wl
from helpers import lm_plan
from test_gpu_lmhead_parity import DEV, run_case

pytestmark = pytest.mark.gpu

SIZES = [
    # rows, vocab, d_model
    (2, 60, 64), (2, 64, 128), (126, 65, 64), (128, 128, 192), (130, 250, 64), (254, 256, 128), (256, 257, 64),
    (258, 320, 64), (384, 321, 128), (386, 900, 64), (640, 1000, 64),
    (130, 5000, 64),    # dL/dH: thin tiles and whole ones, both cut along the vocabulary
    (256, 9000, 576),   # dL/dW: 108 tiles, halved; dL/dH: three tiles in many parts
    (258, 20000, 64),   # 79 whole tiles, halved, and 79 thin ones
    (514, 20000, 64),   # 158 whole tiles: not halved
]


@pytest.mark.parametrize("rows,vocab,d", SIZES)
def test_every_element_around_tile_edges(rows, vocab, d):
    cfg = wl.CONFIGS["numerics_stress"].scaled(n_prompts=1, seq_len=rows // 2, vocab=vocab, group_size=2)
    run_case(cfg, d, label="%dx%dx%d" % (rows, vocab, d), products="library" if rows * vocab * d > 10 ** 8 else "loops")


# more thin tiles than places that are free in the round of the last whole ones: two of them to a place
@pytest.mark.parametrize("rows,vocab,d", [(384, 35840, 64), (512 + 96, 44600, 64)])
def test_thin_tiles_two_to_a_place(rows, vocab, d):
    assert lm_plan(rows, vocab, d)["pairs"] > 0  # no row of this recipe is masked
    cfg = wl.CONFIGS["numerics_stress"].scaled(n_prompts=1, seq_len=rows // 2, vocab=vocab, group_size=2)
    run_case(cfg, d, label="%dx%dx%d" % (rows, vocab, d), products="library")


# results whose rows do not lie on 16 (dL/dW) or 8 bytes (dL/dH) are stored element by element: the same bits, in
# lm_gemm_nt and, where the contraction of dL/dH is cut, for thin tiles or for whole and thin ones, in lm_split_reduce
@pytest.mark.parametrize("rows,vocab,d,cut", [(130, 300, 128, ()), (300, 700, 64, ()), (120, 5000, 64, ("thin",)),
                                              (600, 20000, 128, ("rest", "thin"))])
def test_results_at_odd_pitches_and_offsets(rows, vocab, d, cut):
    g = torch.Generator(device=DEV).manual_seed(rows)
    h = torch.randn(rows, d, generator=g, device=DEV).bfloat16()
    w = (torch.randn(vocab, d, generator=g, device=DEV) * 0.2).bfloat16()
    tokens = torch.randint(0, vocab, (rows,), generator=g, device=DEV)
    adv = torch.randn(rows, generator=g, device=DEV)
    old = grpo.grpo_lmhead_logprobs_fwd(h, w, tokens) + 0.1 * torch.randn(rows, generator=g, device=DEV)
    call = lambda **kw: grpo.grpo_lmhead_loss_fwd_bwd(h, w, tokens, old, adv, **kw)  # noqa: E731
    *_, gh, gw = call()
    ldz = (vocab + 63) // 64 * 64
    plan = lm_plan(int((gh != 0).any(1).sum()), d, ldz, (rows + 255) // 256 * 256 * ldz // 65536)
    assert (plan["s2"] > 1) == bool(cut) and all(plan[kind] > 0 for kind in cut) and ("thin" not in cut or plan["t2"] > 1)
    odd_h = torch.full((rows, d + 1), 7.0, dtype=torch.bfloat16, device=DEV)
    odd_w = torch.full((vocab, d + 3), 7.0, device=DEV)
    call(grad_hidden=odd_h[:, 1:], grad_weight=odd_w[:, 1:d + 1])
    assert torch.equal(odd_h[:, 1:], gh) and torch.equal(odd_w[:, 1:d + 1], gw)
    assert (odd_h[:, 0] == 7).all() and (odd_w[:, 0] == 7).all() and (odd_w[:, d + 1:] == 7).all()
    twice = gw.clone()
    call(grad_weight=twice, accumulate_grad_weight=True)
    call(grad_weight=odd_w[:, 1:d + 1], accumulate_grad_weight=True)
    assert torch.equal(twice, gw + gw) and torch.equal(odd_w[:, 1:d + 1], twice)


# chunks of more than 32768 rows: the rows with a gradient are found through counts per 4096 rows.  One chunk of all rows against the
# default chunks of 10240: log-probs, loss and counters bit for bit, dL/dH to its bf16 rounding (2^-8; a row in another row's place
# is off by its own size), dL/dW to the order of up to 5e4 fp32 sums (their rounding adds up to some sqrt(5e4) 2^-24 = 1.4e-5).
# Gradients everywhere, in a few rows at the edges of those counts, in 64 rows across one, at the end only, and nowhere.
@pytest.mark.parametrize("aux", [False, True])
@pytest.mark.parametrize("rows", [32769, 70001])
def test_gradient_rows_of_large_chunks(rows, aux):
    v, d = 300, 64
    g = torch.Generator(device="cuda").manual_seed(rows)
    h = torch.randn((rows, d), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((v, d), generator=g, device="cuda") * 0.3).to(torch.bfloat16)
    tok = torch.randint(0, v, (rows,), generator=g, device="cuda")
    mask = (torch.rand(rows, generator=g, device="cuda") < 0.8).to(torch.uint8)
    zeros = torch.zeros(rows, device="cuda")
    # the reference is this very call's log-probs: a KL term of a last bit, as against those of the forward alone, has a gradient too
    lp = grpo.grpo_lmhead_loss_aux_fwd_bwd(h, w, tok, zeros, zeros, zeros, mask, kl_coef=0.1, entropy_coef=0.0)[1]
    live = mask.nonzero()[:, 0]
    n = len(live)
    picks = {"all": live, "edges": live[[0, 15, 16, 4095, 4096, 4097, 8191, 20000, n - 1]], "across": live[4064:4128],
             "end": live[n - 4000:], "none": live[:0]}
    for name, pick in picks.items():
        adv = torch.zeros(rows, device="cuda")
        adv[pick] = torch.rand(len(pick), generator=g, device="cuda") + 0.5
        got = []
        for chunk in (10240, rows):
            ws = torch.full((grpo.grpo_lmhead_workspace_bytes_for_chunk(rows, v, d, chunk),), 255, dtype=torch.uint8, device="cuda")
            kw = dict(workspace=ws)
            if aux:  # a gradient where the KL term has one too
                out = grpo.grpo_lmhead_loss_aux_fwd_bwd(h, w, tok, lp + 0.05, lp - 0.1 * (adv != 0), adv, mask, kl_coef=0.1,
                                                        entropy_coef=0.0, **kw)
            else:
                out = grpo.grpo_lmhead_loss_fwd_bwd(h, w, tok, lp + 0.05, adv, mask, **kw)
            got.append(out)
        for a, b in zip(got[0][:-2], got[1][:-2]):
            assert torch.equal(a, b), name
        (ha, wa), (hb, wb) = ([t.float() for t in out[-2:]] for out in got)
        nothing = torch.ones(rows, dtype=torch.bool, device="cuda")
        nothing[pick] = False
        assert bool((hb[nothing] == 0).all()), name
        assert bool(((ha - hb).norm(dim=1) <= ha.norm(dim=1) * 2.0 ** -8).all()), name
        assert float((wa - wb).norm()) <= 1e-4 * float(wa.norm()), name
        assert len(pick) == 0 or float(wb.norm()) > 0
