"""GPU parity of the reward shaping and online filter kernels (sections 3.1, 3.3)."""
import numpy as np
import pytest
import torch

import paper_2505_07291_amd as grpo
from oracle import grpo_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda"


def test_total_rewards():
    g = torch.Generator().manual_seed(2)
    for R in (1, 63, 4096, 100001):
        task = (torch.rand(R, generator=g) < 0.3).float()
        target = torch.tensor([1000, 2000, 3000, 4000], dtype=torch.int32)[torch.randint(0, 4, (R,), generator=g)]
        length = torch.randint(1, 32769, (R,), generator=g, dtype=torch.int32)
        out = grpo.grpo_total_rewards(task.to(DEV), length.to(DEV), target.to(DEV), 3e-4)
        ref = orc.total_rewards(task.numpy(), length.numpy(), target.numpy(), float(np.float32(3e-4)))
        got = out.cpu().numpy().astype(np.float64)
        # one product and one difference in fp32 against fp64
        assert np.max(np.abs(got - ref)) <= 2.0 ** -22 * np.maximum(1.0, np.abs(ref)).max()
    assert grpo.grpo_total_rewards(task[:0].to(DEV), length[:0].to(DEV), target[:0].to(DEV), 3e-4).numel() == 0


def test_filter_groups_bit_exact():
    g = torch.Generator().manual_seed(3)
    for G, n in ((16, 256), (4, 5000), (64, 33), (1, 10), (100, 1500)):
        R = (torch.rand(G * n, generator=g) < 0.15).float()
        R[:G] = 1.0
        keep, kept, n_kept, rk = grpo.grpo_filter_groups(R.to(DEV), group_size=G)
        torch.cuda.synchronize()
        rkeep, rkept, rn, rrk = orc.filter_groups(R.numpy(), group_size=G)
        assert np.array_equal(keep.cpu().numpy(), rkeep) and int(n_kept) == rn
        assert np.array_equal(kept.cpu().numpy(), rkept)
        assert np.array_equal(rk.cpu().numpy(), rrk)
    sizes = [3, 1, 16, 0, 70, 5, 2]
    off = torch.tensor(np.concatenate([[0], np.cumsum(sizes)]), dtype=torch.int32)
    R = torch.randint(0, 3, (int(off[-1]),), generator=g).float() * 0.5
    R[off[5]:off[6]] = 0.5                                    # a constant group
    keep, kept, n_kept, rk = grpo.grpo_filter_groups(R.to(DEV), group_offsets=off.to(DEV))
    rkeep, rkept, rn, rrk = orc.filter_groups(R.numpy(), group_offsets=off.numpy())
    assert np.array_equal(keep.cpu().numpy(), rkeep) and int(n_kept) == rn
    assert np.array_equal(kept.cpu().numpy(), rkept) and np.array_equal(rk.cpu().numpy(), rrk)
    # no groups at all
    keep, kept, n_kept, rk = grpo.grpo_filter_groups(R[:0].to(DEV), group_size=4)
    assert int(n_kept) == 0


def test_reward_chain_feeds_the_advantages():
    """total reward -> filter -> advantages of the kept groups, as the trainer would chain them."""
    g = torch.Generator().manual_seed(4)
    G, n = 16, 64
    task = (torch.rand(G * n, generator=g) < 0.2).float()
    target = torch.full((G * n,), 2000, dtype=torch.int32)
    length = torch.randint(500, 4000, (G * n,), generator=g, dtype=torch.int32)
    length[:G] = 2000
    task[:G] = 0.0                                            # equal total rewards: filtered out
    rew = grpo.grpo_total_rewards(task.to(DEV), length.to(DEV), target.to(DEV), 3e-4)
    keep, kept, n_kept, _ = grpo.grpo_filter_groups(rew, group_size=G)
    adv, _ = grpo.grpo_group_advantages(rew, group_size=G)
    torch.cuda.synchronize()
    assert int(keep[0]) == 0 and int(n_kept) == n - 1
    a = adv.cpu().numpy().reshape(n, G)
    assert not a[0].any() and np.all(np.any(a[1:] != 0, axis=1))


# one lane to a group up to 1024 groups of up to 64 and 16384 rollouts, a wavefront to a group beyond: both
# sides of each limit, and of the 64 groups of a wavefront
@pytest.mark.parametrize("G,n", [(16, 1024), (16, 1025), (64, 256), (64, 257), (64, 1024), (65, 252), (17, 963), (17, 964),
                                 (1, 1024), (7, 63), (7, 64), (7, 65), (2, 961)])
def test_filter_groups_around_its_limits(G, n):
    g = torch.Generator().manual_seed(G * 10000 + n)
    R = (torch.rand(G * n, generator=g) < 0.2 / G ** 0.5).float()
    if G > 1:
        R[-1] = float("nan")                                  # differs from the others, whatever they are
    keep, kept, n_kept, rk = grpo.grpo_filter_groups(R.to(DEV), group_size=G)
    torch.cuda.synchronize()
    rkeep, rkept, rn, rrk = orc.filter_groups(R.numpy(), group_size=G)
    assert np.array_equal(keep.cpu().numpy(), rkeep) and int(n_kept) == rn
    assert np.array_equal(kept.cpu().numpy(), rkept) and np.array_equal(rk.cpu().numpy(), rrk)


@pytest.mark.parametrize("R,size", [(3, 4), (1, 16), (5, 0)])
def test_filter_without_a_whole_group_flags_nobody(R, size):
    """Fewer rewards than a group takes, or no group size: there is no group, and no rollout is flagged as
    kept, whatever the memory of the flags held before."""
    dirt = [torch.full((512,), 255, dtype=torch.uint8, device=DEV) for _ in range(4096)]
    torch.cuda.synchronize()
    del dirt                                                  # the allocator hands these blocks out again
    keep, kept, n_kept, rk = grpo.grpo_filter_groups(torch.rand(R, device=DEV), group_size=size)
    torch.cuda.synchronize()
    assert keep.numel() == 0 and kept.numel() == 0 and int(n_kept) == 0
    assert rk.tolist() == [0] * R


def test_packed_layout_with_decreasing_offsets():
    """Offsets that decrease or leave the batch: no weight is infinite, a row either has the weight of a rollout
    whose range it is in or none, and rows away from the fault are what they would be without it."""
    cu = torch.tensor([0, 10, 5, 20, 20, 900, 40, 1000, 5000], dtype=torch.int64)
    n = 1024
    w, rot = grpo.grpo_packed_layout(cu.to(DEV), n, True)
    torch.cuda.synchronize()
    w, rot, c = w.cpu().numpy(), rot.cpu().numpy(), cu.numpy().clip(0, n)
    assert np.isfinite(w).all() and np.array_equal(w == 0, rot == -1)
    t = np.flatnonzero(rot >= 0)
    b, e = c[rot[t]], c[rot[t] + 1]
    assert np.all((b <= t) & (t < e)) and np.array_equal(w[t], (1.0 / (e - b)).astype(np.float32))
    assert np.all(rot[:5] == 0) and np.all(rot[10:20] == 2) and np.all(rot[20:40] == 4) and np.all(rot[1000:] == 7)


# a wavefront looks 64 of the R + 1 offsets up at once (65: a second round, 4097: a third), for 256 rows; a
# workgroup has four wavefronts, and the grid 4096 workgroups
@pytest.mark.parametrize("R", [1, 62, 63, 64, 4095, 4096, 9000])
def test_packed_layout_search(R):
    g = torch.Generator().manual_seed(R)
    for n in (1, 255, 256, 257, 1024, 1025, 4099, 70001):
        lead, trail = (n // 10, n // 7) if n > 255 else (0, 0)  # rows before and after the rollouts are nobody's
        cu = torch.randint(lead, n - trail + 1, (R + 1,), generator=g).sort().values
        cu[0] = lead                                          # (R above n: most rollouts are empty)
        for sample_level in (True, False):
            w, rot = grpo.grpo_packed_layout(cu.to(DEV), n, sample_level)
            torch.cuda.synchronize()
            w_ref, rot_ref = orc.packed_layout(cu.numpy(), n, sample_level)
            assert np.array_equal(rot.cpu().numpy(), rot_ref), (R, n)
            assert np.array_equal(w.cpu().numpy(), w_ref), (R, n)


def test_packed_layout_of_more_rows_than_the_grid_takes_at_once():
    n, R = 4096 * 1024 + 300, 3000
    cu = torch.randint(0, n + 1, (R + 1,), generator=torch.Generator().manual_seed(5)).sort().values
    w, rot = grpo.grpo_packed_layout(cu.to(DEV), n, True)
    torch.cuda.synchronize()
    w_ref, rot_ref = orc.packed_layout(cu.numpy(), n, True)
    assert np.array_equal(rot.cpu().numpy(), rot_ref) and np.array_equal(w.cpu().numpy(), w_ref)


# advantages and their tokens in one launch: 16 lanes to a group of up to 16 rollouts (64 groups at once, up to
# four rounds), 64 to a larger one (16 at once); at most 1024 rollouts; 4096 tokens to a workgroup.  Both sides of
# each limit.
@pytest.mark.parametrize("G,n_groups", [(16, 1), (16, 63), (16, 64), (1, 256), (1, 257), (4, 255), (4, 256), (4, 257), (15, 65),
                                        (17, 1), (17, 16), (17, 17), (17, 60), (64, 16), (64, 17), (100, 10), (1000, 1),
                                        (1024, 1), (1025, 1)])
@pytest.mark.parametrize("ddof", [0, 1])
def test_advantages_of_equal_groups_with_tokens(G, n_groups, ddof):
    g = torch.Generator().manual_seed(1000 * G + n_groups)
    R = G * n_groups
    rewards = (torch.randint(0, 5, (R,), generator=g).float() * 0.25)
    rewards[-G:] = 0.5                                        # a group without signal
    ref = orc.group_advantages(rewards.numpy(), group_size=G, eps_std=float(np.float32(1e-6)), ddof=ddof)
    for n in (1, 1024, 4095, 4096, 4097, 20000):
        rot = torch.randint(0, R, (n,), generator=g, dtype=torch.int32)
        bad = torch.rand(n, generator=g) < 0.05
        rot[bad] = torch.tensor([-1, R, 10 ** 9, -10 ** 9], dtype=torch.int32)[torch.randint(0, 4, (int(bad.sum()),), generator=g)]
        adv, adv_tok = grpo.grpo_group_advantages(rewards.to(DEV), group_size=G, ddof=ddof, rollout_of_token=rot.to(DEV))
        torch.cuda.synchronize()
        a, t = adv.cpu().numpy(), adv_tok.cpu().numpy()
        assert np.max(np.abs(a - ref)) <= 2e-6 * max(1.0, np.max(np.abs(ref))) and not a[-G:].any()
        assert np.isnan(t[bad.numpy()]).all()
        assert np.array_equal(t[~bad.numpy()], a[rot[~bad].numpy()])
