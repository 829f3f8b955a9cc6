"""The binding's native part: what it takes gives the bits of the general path, what it declines goes there, and what
was refused stays refused with the same exception."""
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2505_07291_amd as grpo
from paper_2505_07291_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(n=48, v=520, dtype=torch.bfloat16, seed=3):
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device=DEV)  # noqa: E731
    logits = (rnd(n, v) * 3).to(dtype)
    tokens = torch.randint(0, v, (n,), generator=g, device=DEV)
    mask = (torch.rand(n, generator=g, device=DEV) < 0.7).to(torch.uint8)
    old = grpo.grpo_logprobs_fwd(logits, tokens) + 0.1 * rnd(n)
    rewards = (torch.rand(32, generator=g, device=DEV) < 0.5).float()
    rewards[8 * (seed % 4):8 * (seed % 4) + 8] = 1.0  # a group without a signal
    return dict(logits=logits, tokens=tokens, mask=mask, old=old, ref=old + 0.05 * rnd(n), adv=rnd(n),
                grad=torch.empty_strided(logits.shape, logits.stride(), dtype=dtype, device=DEV),
                rewards=rewards,
                lengths=torch.randint(1, 99, (32,), generator=g, device=DEV, dtype=torch.int32),
                target=torch.randint(1, 99, (32,), generator=g, device=DEV, dtype=torch.int32),
                cu=torch.arange(0, 33, device=DEV) * 2 + seed - 3, rollout=torch.arange(n, device=DEV, dtype=torch.int32) % 32)


CALLS = {
    "grpo_total_rewards": lambda s, **kw: grpo.grpo_total_rewards(s["rewards"], s["lengths"], s["target"], 3e-4, **kw),
    "grpo_filter_groups": lambda s, **kw: grpo.grpo_filter_groups(s["rewards"], group_size=8, **kw),
    "grpo_packed_layout": lambda s, **kw: grpo.grpo_packed_layout(s["cu"], 70, True, **kw),
    "grpo_group_advantages": lambda s, **kw: grpo.grpo_group_advantages(s["rewards"], 8, rollout_of_token=s["rollout"], **kw),
    "grpo_group_advantages alone": lambda s, **kw: grpo.grpo_group_advantages(s["rewards"], group_size=16, ddof=1, **kw),
    "grpo_logprobs_fwd": lambda s, **kw: grpo.grpo_logprobs_fwd(s["logits"], s["tokens"], s["mask"], 0.7, **kw),
    "grpo_loss_fwd_bwd": lambda s, **kw: grpo.grpo_loss_fwd_bwd(
        s["logits"], s["tokens"], s["old"], s["adv"], s["mask"], grad_logits=s["grad"], **kw),
    "grpo_loss_fwd_bwd default": lambda s, **kw: grpo.grpo_loss_fwd_bwd(s["logits"], s["tokens"], s["old"], s["adv"], s["mask"], **kw),
    "grpo_loss_fwd_bwd in place": lambda s, **kw: grpo.grpo_loss_fwd_bwd(
        s["logits"].clone(), s["tokens"], s["old"], s["adv"], inplace=True, **kw),
    "grpo_loss_aux_fwd_bwd default": lambda s, **kw: grpo.grpo_loss_aux_fwd_bwd(
        s["logits"][:, :511], s["tokens"] // 2, s["old"], None, s["adv"], s["mask"], want_entropy=False, **kw),
    "grpo_loss_aux_fwd_bwd in place": lambda s, **kw: grpo.grpo_loss_aux_fwd_bwd(
        s["logits"].clone(), s["tokens"], s["old"], s["ref"], s["adv"], s["mask"], kl_coef=0.1, inplace=True, **kw),
    "grpo_loss_aux_fwd_bwd": lambda s, **kw: grpo.grpo_loss_aux_fwd_bwd(
        s["logits"], s["tokens"], s["old"], s["ref"], s["adv"], None, 0.1, 0.3, 5, 1, 0.001, 1e-4, 17, grad_logits=s["grad"], **kw),
}


def flat(out):
    return [None if t is None else t.clone() for t in (out if isinstance(out, tuple) else (out,))]


class Seen(TorchDispatchMode):
    ops = 0

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        Seen.ops += 1
        return func(*args, **(kwargs or {}))


class Spy:
    """Stands for the native part and notes which of its functions took a call."""

    def __init__(self, native):
        self.native, self.taken = native, []

    def __getattr__(self, name):
        def call(*args):
            out = getattr(self.native, name)(*args)
            self.taken.append((name, out is not None))
            return out
        return call


@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_same_results_as_the_general_path(name, dtype, monkeypatch):
    s, fn = inputs(dtype=dtype), name.split()[0][5:]
    spy = Spy(binding._fast)
    monkeypatch.setattr(binding, "_fast", spy)
    fast = flat(CALLS[name](s))
    assert spy.taken == [(fn, True)]
    general = flat(CALLS[name](s, stream=torch.cuda.current_stream()))  # a stream of the caller's: not asked at all
    assert spy.taken == [(fn, True)]
    Seen.ops = 0
    with Seen():  # a mode that wants to see the allocations: declined
        seen = flat(CALLS[name](s))
    assert spy.taken == [(fn, True), (fn, False)] and Seen.ops > 0
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.inference_mode(), torch.autocast("cuda"):
        other = flat(CALLS[name](s))
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for a, b, c, d in zip(fast, general, seen, other):
        assert (a is None) == (b is None) == (c is None) == (d is None)
        if a is not None:
            assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device
            assert torch.equal(a, b) and torch.equal(a, c) and torch.equal(a, d)


def refill(s, new):
    """Other values in the same tensors, by work on the current stream."""
    for k, t in s.items():
        t.copy_(new[k])


def test_calls_are_made_on_the_current_stream(monkeypatch):
    """The inputs arrive on a side stream behind a wait of some milliseconds: a call made on any other stream would
    see those of before."""
    s, first, later = inputs(), inputs(), inputs(seed=4)
    before = {name: flat(call(first)) for name, call in CALLS.items()}
    want = {name: flat(call(later)) for name, call in CALLS.items()}
    for name in CALLS:
        assert any(a is not None and not torch.equal(a, b) for a, b in zip(before[name], want[name])), name
    spy, side = Spy(binding._fast), torch.cuda.Stream()
    monkeypatch.setattr(binding, "_fast", spy)
    for name, call in CALLS.items():
        refill(s, first)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(10 ** 7)
            refill(s, later)
            got = flat(call(s))
        torch.cuda.synchronize()
        for a, b in zip(got, want[name]):
            assert (a is None and b is None) or torch.equal(a, b), name
    assert len(spy.taken) == len(CALLS) and all(took for _, took in spy.taken)


def test_captured_calls(monkeypatch):
    """Every call, its outputs allocated by the native part, in one captured graph: replays over changing inputs, with
    eager work between them, give the eager bits."""
    spy = Spy(binding._fast)
    s = inputs()
    run = lambda: {name: call(s) for name, call in CALLS.items()}  # noqa: E731
    run()  # first uses: attributes of the kernels, the queue's workspace
    torch.cuda.synchronize()
    monkeypatch.setattr(binding, "_fast", spy)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        outs = run()
    assert len(spy.taken) == len(CALLS) and all(took for _, took in spy.taken)
    torch.cuda.synchronize()
    for seed in (3, 4, 5, 4):
        refill(s, inputs(seed=seed))
        # (calls that share the caller's gradient tensor leave the last one's in it)
        want = {name: flat(out) for name, out in run().items()}
        torch.cuda.synchronize()
        for out in outs.values():
            for t in out if isinstance(out, tuple) else (out,):
                if t is not None:
                    t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for name, out in outs.items():
            for a, b in zip(flat(out), want[name]):
                assert (a is None and b is None) or torch.equal(a, b), "%s, seed %d" % (name, seed)


class Sub(torch.Tensor):
    pass


def test_declined_and_refused_calls():
    s = inputs()
    assert binding._fast.total_rewards(s["rewards"].as_subclass(Sub), s["lengths"], s["target"], 3e-4) is None
    assert binding._fast.total_rewards(s["rewards"].cpu(), s["lengths"].cpu(), s["target"].cpu(), 3e-4) is None
    assert binding._fast.total_rewards(s["rewards"], s["lengths"], s["target"], torch.tensor(3e-4)) is None
    assert binding._fast.filter_groups(s["rewards"], True) is None
    assert torch.equal(CALLS["grpo_total_rewards"](s),
                       grpo.grpo_total_rewards(s["rewards"].as_subclass(Sub), s["lengths"], s["target"], torch.tensor(3e-4)))
    for change, call in ((dict(lengths=s["lengths"].long()), "grpo_total_rewards"), (dict(target=s["target"][:-1]), "grpo_total_rewards"),
                         (dict(rollout=s["rollout"].long()), "grpo_group_advantages"), (dict(cu=s["cu"].int()), "grpo_packed_layout"),
                         (dict(mask=s["mask"].float()), "grpo_logprobs_fwd"), (dict(adv=s["adv"].repeat(2)[::2]), "grpo_loss_fwd_bwd"),
                         (dict(grad=s["grad"].float()), "grpo_loss_fwd_bwd"), (dict(old=s["old"].cpu()), "grpo_loss_fwd_bwd"),
                         (dict(logits=s["logits"].half()), "grpo_loss_aux_fwd_bwd")):
        with pytest.raises(ValueError):
            CALLS[call](dict(s, **change))
    for bad in (lambda: grpo.grpo_filter_groups(s["rewards"], group_size=5),            # sizes that leave rollouts over
                lambda: grpo.grpo_group_advantages(s["rewards"], 5), lambda: grpo.grpo_logprobs_fwd(s["logits"], s["tokens"], None, 0.0),
                lambda: grpo.grpo_loss_fwd_bwd(s["logits"], s["tokens"], s["old"], s["adv"], s["mask"], 0.2, 0.2, 1.1, grad_logits=s["grad"]),
                lambda: grpo.grpo_group_advantages(s["rewards"], 8, ddof=2)):
        with pytest.raises(grpo.GrpoError):
            bad()
