"""Row widths and batch sizes at which the row kernels change what they do, against the fp64 oracle
(log-probs, loss and counters of every row, gradients of sampled rows, in place as well): tolerances and
comparison are those of the other shapes (run_shape_case)."""
import numpy as np
import pytest
import torch

import paper_2505_07291_amd as grpo
import paper_2505_07291_amd.workloads as wl
from test_gpu_aux_parity import run_aux_shape_case
from test_gpu_lmhead_parity import run_case
from test_gpu_parity import run_shape_case

pytestmark = pytest.mark.gpu


def sampled(rows, seed):
    rng = np.random.default_rng(seed)
    return np.unique(np.concatenate([np.arange(min(rows, 6)), np.arange(max(0, rows - 6), rows),
                                     rng.choice(rows, size=min(rows, 40), replace=False)]))


# the streaming kernel works in batches of 2048 vectors through two buffers: an even and an odd number
# of whole batches, one vector more, and one less; ragged, so that no resident kernel takes them
@pytest.mark.parametrize("dtype,epv", [("bf16", 8), ("f32", 4)])
@pytest.mark.parametrize("vectors", [10 * 2048, 10 * 2048 + 1, 11 * 2048, 9 * 2048 - 1])
def test_streamed_rows_around_whole_batches(dtype, epv, vectors):
    vocab = vectors * epv + epv - 1
    run_shape_case(dtype, vocab, vocab + 1, 600, grad_rows=sampled(600, vectors))


# narrow rows: at most one row for each workgroup, up to eight, and more (through the queue)
@pytest.mark.parametrize("rows", [1, 7, 2048, 2049, 8192, 8193, 16384, 16385])
def test_narrow_rows_strided_and_queued(rows):
    run_shape_case("f32", 1024, 1024, rows, grad_rows=sampled(rows, rows))


# ragged rows that stay in registers: the last vector of a width, and the first one past it
@pytest.mark.parametrize("dtype,epv", [("bf16", 8), ("f32", 4)])
@pytest.mark.parametrize("vectors", [10240, 26 * 512 - 1, 26 * 512, 32 * 512 - 1, 32 * 512])
def test_ragged_rows_around_the_resident_widths(dtype, epv, vectors):
    vocab = vectors * epv + 1
    run_shape_case(dtype, vocab, (vectors + 1) * epv, 300, grad_rows=sampled(300, vectors))


# the head's rows are taken by one kernel up to 32768 tokens, by the walk and the gather beyond; groups
# of 16 rows, the last one whole, of one row, and short of one
@pytest.mark.parametrize("prompts,seq", [(1, 1), (2, 33), (8, 256), (8, 257)])
def test_head_rows_taken_by_either_path(prompts, seq):
    cfg = wl.CONFIGS["qwen_short"].scaled(n_prompts=prompts, seq_len=seq, vocab=40, group_size=16)
    run_case(cfg, 64, label="N=%d" % cfg.n_tokens)


# partials per row merged by 16 lanes (one, and all of their 192 tiles) and by 64 (one tile more, and more
# tiles than their registers hold)
@pytest.mark.parametrize("vocab", [256, 192 * 256, 192 * 256 + 1, 768 * 256 + 300])
def test_head_partials_of_few_and_many_tiles(vocab):
    cfg = wl.CONFIGS["qwen_short"].scaled(n_prompts=1, seq_len=5, vocab=vocab, group_size=4)
    run_case(cfg, 64, label="V=%d" % vocab)


# rows strided over the grid, several rounds of it, where workgroups share a CU and where each has one to
# itself, or from the queue, the last four in batches long enough for two increments at once: every row is taken once, whatever
# workgroup takes it
@pytest.mark.parametrize("dtype,vocab,rows", [("f32", 1000, 9000), ("bf16", 8192, 5000), ("bf16", 50304, 1300),
                                              ("bf16", 100352, 1030), ("f32", 50257, 700), ("bf16", 8192, 14000),
                                              ("bf16", 16384, 6000), ("bf16", 107008, 2500), ("f32", 50257, 2400)])
def test_strided_rows_equal_queued_rows(dtype, vocab, rows):
    g = torch.Generator(device="cuda").manual_seed(vocab)
    pitch = (vocab + 7) // 8 * 8
    logits = torch.randn((rows, pitch), generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    tokens = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
    mask = (torch.rand(rows, generator=g, device="cuda") < 0.6).to(torch.uint8)
    out = torch.full((rows,), 3.0, device="cuda")
    grpo.grpo_logprobs_fwd(logits[:, :vocab], tokens, mask, logprobs_out=out, use_queue=False)
    want = grpo.grpo_logprobs_fwd(logits[:, :vocab], tokens, mask)
    torch.cuda.synchronize()
    assert torch.equal(out, want) and bool((out[mask == 0] == 0).all()) and bool((out[mask != 0] < 0).all())


# the same widths with the auxiliary terms, which have code of their own at every stage of a row; per-token
# weights in every other case; each workgroup takes rows in turn
@pytest.mark.parametrize("dtype,epv", [("bf16", 8), ("f32", 4)])
@pytest.mark.parametrize("vectors", [10240, 26 * 512 - 1, 26 * 512, 32 * 512 - 1, 32 * 512])
def test_aux_ragged_rows_around_the_resident_widths(dtype, epv, vectors):
    run_aux_shape_case(dtype, vectors * epv + epv - 1, (vectors + 1) * epv, 400, weights=vectors % 2 == 0)


# streamed rows: an even and an odd number of batches, whole and with a vector more; more rows than
# workgroups, so that a row's gradient pass loads the next row
@pytest.mark.parametrize("dtype,epv,vectors", [("bf16", 8, 10 * 2048), ("bf16", 8, 9 * 2048 - 1), ("f32", 4, 10 * 2048 + 1),
                                               ("f32", 4, 11 * 2048)])
def test_aux_streamed_rows_around_whole_batches(dtype, epv, vectors):
    vocab = vectors * epv + 1
    run_aux_shape_case(dtype, vocab, (vectors + 1) * epv, 700, weights=vectors % 2 == 0)


# up to 1024 rows of up to 1024 vectors the row kernel counts the rows itself and writes the header; with one row
# more, masked, grpo_prepare does: the same bits, counters and error word, with and without a bad token id
@pytest.mark.parametrize("aux", [False, True])
@pytest.mark.parametrize("dtype,vocab", [(torch.bfloat16, 1000), (torch.bfloat16, 8191), (torch.float32, 4096), (torch.float32, 4100)])
@pytest.mark.parametrize("rows,bad", [(1024, None), (1024, 1023), (1024, 5)])
def test_rows_counted_by_the_row_kernel(aux, dtype, vocab, rows, bad):
    g = torch.Generator(device="cuda").manual_seed(vocab)
    pitch = (vocab + 7) // 8 * 8
    logits = (torch.randn(rows + 1, pitch, generator=g, device="cuda") * 3).to(dtype)[:, :vocab]
    tokens = torch.randint(0, vocab, (rows + 1,), generator=g, device="cuda")
    old, adv, ref = (torch.randn(rows + 1, generator=g, device="cuda") for _ in range(3))
    mask = (torch.rand(rows + 1, generator=g, device="cuda") < 0.7).to(torch.uint8)
    weights = torch.rand(rows + 1, generator=g, device="cuda") * (torch.rand(rows + 1, generator=g, device="cuda") < 0.9)
    mask[rows] = 0
    if bad is not None:
        tokens[bad], mask[bad], weights[bad] = vocab, 1, 0.5
    for denom in (0.0, 777.0):
        got = []
        for n in (rows, rows + 1):
            ws = torch.full((grpo.grpo_workspace_bytes(n),), 255, dtype=torch.uint8, device="cuda")
            grad = torch.full((n, pitch), 7.0, dtype=dtype, device="cuda")[:, :vocab]
            kw = dict(denom=denom, grad_logits=grad, workspace=ws)
            if aux:
                out = grpo.grpo_loss_aux_fwd_bwd(logits[:n], tokens[:n], old[:n], ref[:n], adv[:n], mask[:n], kl_coef=0.1,
                                                 entropy_coef=0.01, token_weights=weights[:n], **kw)
            else:
                out = grpo.grpo_loss_fwd_bwd(logits[:n], tokens[:n], old[:n], adv[:n], mask[:n], **kw)
            error = grpo.grpo_workspace_error(ws)
            assert error == (0 if bad is None else 1)
            got.append([t[:rows] if t.dim() > 0 and t.shape[0] == n else t for t in out])
        for a, b in zip(*got):
            assert torch.equal(a, b)


# gradient rows that begin with a 128-byte line, or anywhere inside one: the resident kernels may then hold a row up to seven
# vectors further back, the streaming one turns its lanes, and both sum in the same order: the same bits, nothing written
# outside the rows.  Every resident width, whole and ragged rows, the last widths that leave room for it and the first that
# do not; streamed ragged rows (those of more than 16384 vectors).  At most a row to a workgroup, where only the resident
# kernels of wide rows do so.
@pytest.mark.parametrize("aux", [False, True])
@pytest.mark.parametrize("dtype,epv", [(torch.bfloat16, 8), (torch.float32, 4)])
@pytest.mark.parametrize("vectors", [1, 5, 249, 250, 1017, 1018, 4000, 6649, 8185, 8186, 10233, 13305, 16377, 16378, 19449,
                                     22521, 22522])
def test_rows_that_begin_inside_a_line(aux, dtype, epv, vectors):
    rows = 23
    for tail in (0, epv - 1):
        vocab = vectors * epv + tail
        g = torch.Generator(device="cuda").manual_seed(vocab)
        z = (torch.randn(rows, vocab, generator=g, device="cuda") * 3).to(dtype)
        z[1, : vocab // 2] = float("-inf")
        tokens = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
        tokens[0], tokens[1], tokens[2] = 0, vocab - 1, min(vocab - 1, 3 * epv)
        old, adv, ref = (torch.randn(rows, generator=g, device="cuda") for _ in range(3))
        mask = (torch.rand(rows, generator=g, device="cuda") < 0.7).to(torch.uint8)
        mask[:4] = 1
        want = None
        for start, apart in ((0, 8), (0, 1), (3, 8), (5, 3), (7, 7)):   # of the first row, between rows: in vectors mod 8
            pitch = ((vectors + 1 + 7) // 8 * 8 + apart % 8) * epv
            size = rows * pitch + 8 * epv + pitch
            bufs = [torch.full((size,), 3.0, dtype=dtype, device="cuda") for _ in range(2)]
            views = [b[start * epv:].as_strided((rows, vocab), (pitch, 1)) for b in bufs]
            views[0].copy_(z)
            for b in bufs:
                assert b.data_ptr() % 128 == 0
            if aux:
                out = grpo.grpo_loss_aux_fwd_bwd(views[0], tokens, old, ref, adv, mask, kl_coef=0.1, entropy_coef=0.01,
                                                 grad_logits=views[1])
            else:
                out = grpo.grpo_loss_fwd_bwd(views[0], tokens, old, adv, mask, grad_logits=views[1])
            got = [views[1].clone()] + [t for t in out[:-1]]
            views[1].fill_(3.0)
            assert bool((bufs[1] == 3.0).all()), "written outside the rows"
            if want is None:
                want = got
            for a, b in zip(got, want):
                assert torch.equal(a.nan_to_num(nan=77.0), b.nan_to_num(nan=77.0)), (vocab, start, apart)


# the same with several rows to a workgroup, from the queue, and different places in a line from one row to the next: a
# workgroup refills its registers in front of and behind what the row before had, lanes turn between rows.  Two masks: most
# rows live, and few, so that masked rows are filled behind the last live ones.  Rows enough for every kernel by its workgroups
# to a CU, more than eight rounds of those that take several narrow rows at once.
@pytest.mark.parametrize("aux", [False, True])
@pytest.mark.parametrize("dtype,epv", [(torch.bfloat16, 8), (torch.float32, 4)])
@pytest.mark.parametrize("vectors", [200, 800, 1016, 1300, 2600, 4088, 6648, 8184, 8185, 10232, 10233, 13304, 13305, 16376,
                                     16377, 19448, 19449, 22520])
def test_several_rows_that_begin_inside_a_line(aux, dtype, epv, vectors):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tail = epv - 3 if vectors % 2 else 0
    per_cu = 8 if vectors <= 1024 else 4 if vectors <= 4096 else 2 if vectors <= 8192 else 1  # streamed: 2, of four rounds' rows
    rows = (8 if vectors * 16 < 32768 else 4 if per_cu == 1 else 3) * per_cu * cus + 37
    vocab = vectors * epv + tail
    g = torch.Generator(device="cuda").manual_seed(vocab)
    pitches = [((vectors + 1 + 7) // 8 * 8 + apart) * epv for apart in (0, 1, 3, 4)]
    z = torch.empty((rows, vocab), dtype=dtype, device="cuda")
    for a in range(0, rows, 256):
        z[a:a + 256] = torch.randn((len(z[a:a + 256]), vocab), generator=g, device="cuda") * 3
    tokens = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
    tokens[::3], tokens[1::5] = 0, vocab - 1
    old, adv, ref = (torch.randn(rows, generator=g, device="cuda") for _ in range(3))
    old -= 12
    bufs = [torch.empty(rows * pitches[-1] + 16 * epv, dtype=dtype, device="cuda") for _ in range(2)]
    for share in (0.7, 0.15):
        mask = (torch.rand(rows, generator=g, device="cuda") < share).to(torch.uint8)
        want = None
        for pitch, start in zip(pitches, (0, 3, 0, 7)):
            for b in bufs:
                b.fill_(3.0)
                assert b.data_ptr() % 128 == 0
            views = [b[start * epv:].as_strided((rows, vocab), (pitch, 1)) for b in bufs]
            views[0].copy_(z)
            ws = torch.full((grpo.grpo_workspace_bytes(rows),), 255, dtype=torch.uint8, device="cuda")
            kw = dict(grad_logits=views[1], workspace=ws)
            if aux:
                out = grpo.grpo_loss_aux_fwd_bwd(views[0], tokens, old, ref - 12, adv, mask, kl_coef=0.1, entropy_coef=0.01, **kw)
            else:
                out = grpo.grpo_loss_fwd_bwd(views[0], tokens, old, adv, mask, **kw)
            got = [views[1].clone()] + list(out[:-1])
            views[1].fill_(3.0)
            assert bool((bufs[1] == 3.0).all()), "written outside the rows"
            if want is None:
                want = got
                assert bool((got[0][mask == 0] == 0).all()) and bool(got[0].isfinite().all())
            for a, b in zip(got, want):
                assert torch.equal(a, b), (vocab, start, pitch, share)


# masked rows behind the live ones, filled in front of a workgroup's last live row or behind it: batches on either side of each
# condition of the rule, by the live ones of their rows, in each kind of kernel (one, two and four workgroups to a CU, rows
# with LDS slots, a streamed remainder, streamed; 600 and 700 rows take the kernels for few rounds).  Every row's values are those it has in a batch without an order (as many
# rows as CUs at most), masked rows are zeros, and nothing is written outside the rows.
@pytest.mark.parametrize("aux", [False, True])
@pytest.mark.parametrize("dtype,vocab,rows", [("bf16", 152064, 700), ("bf16", 81925, 700), ("bf16", 200064, 600), ("bf16", 65536, 1100),
                                              ("bf16", 16384, 1300), ("f32", 50304, 700), ("bf16", 300000, 520), ("bf16", 152069, 1100),
                                              ("bf16", 71616, 411), ("f32", 65533, 768), ("bf16", 240000, 700), ("f32", 75008, 769),
                                              ("bf16", 17470, 1300), ("bf16", 131081, 2100)])
def test_masked_rows_before_and_behind_live_ones(dtype, vocab, rows, aux):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator(device="cuda").manual_seed(vocab)
    pitch = (vocab + 7) // 8 * 8
    z = torch.empty((rows, pitch), dtype=dt, device="cuda")
    for a in range(0, rows, 100):
        z[a:a + 100] = torch.randn((len(z[a:a + 100]), pitch), generator=g, device="cuda") * 3
    tokens = torch.randint(0, vocab, (rows,), generator=g, device="cuda")
    old = -12 + torch.randn(rows, generator=g, device="cuda")
    adv, ref = (torch.randn(rows, generator=g, device="cuda") for _ in range(2))
    order = torch.randperm(rows, generator=torch.Generator().manual_seed(rows))

    def step(part, mask):
        n = len(tokens[part])
        grad = torch.full((n, pitch), 3.0, dtype=dt, device="cuda")
        ws = torch.full((grpo.grpo_workspace_bytes(n),), 255, dtype=torch.uint8, device="cuda")
        kw = dict(denom=50.0, grad_logits=grad[:, :vocab], workspace=ws)
        if aux:
            out = grpo.grpo_loss_aux_fwd_bwd(z[part][:, :vocab], tokens[part], old[part], ref[part], adv[part], mask[part],
                                             kl_coef=0.1, entropy_coef=0.01, **kw)
        else:
            out = grpo.grpo_loss_fwd_bwd(z[part][:, :vocab], tokens[part], old[part], adv[part], mask[part], **kw)
        assert bool((grad[:, vocab:] == 3.0).all()), "written outside the rows"
        return [grad[:, :vocab]] + [t for t in out[1:-1] if t.shape[0] == n]

    edges = {cus * 5, cus * 5 + 1, cus * 8, cus * 8 + 1}  # five rows on four workgroups of four to a CU, four to one of two
    for live in sorted({0, 1, 40, rows // 5, max(0, rows - 2 * cus - 1), rows * 5 // 8, rows - 1} | {e for e in edges if e < rows}):
        mask = torch.zeros(rows, dtype=torch.uint8)
        mask[order[:live]] = 1
        mask = mask.to("cuda")
        whole = step(slice(0, rows), mask)
        assert bool((whole[0][mask == 0] == 0).all())
        for a in range(0, rows, cus):
            for t, part in zip(whole, step(slice(a, a + cus), mask)):
                assert torch.equal(t[a:a + cus], part), (live, a)
