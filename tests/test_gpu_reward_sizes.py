"""Reward statistics on both sides of each choice: ranks up to 256 seeds and an LDS sort past that, the
finiteness check inside the statistics launch up to 16384 rewards and as a pass of its own past that, for many groups or
when an output lies over the rewards. Orders are compared exactly with the oracle's stable sort."""
import numpy as np
import pytest
import torch

from oracle import dit_oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    from paper_2606_19004_amd import ditstep
    return ditstep


def outputs(g, n, k):
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(device="cuda")
    return dict(mean=torch.empty(g, **f32), std=torch.empty(g, **f32), adv=torch.empty(g, n, **f32),
                order=torch.full((g, n), -7, **i32), selected=torch.full((g, k), -7, **i32))


def check(r, out, k):
    want = O.group_reward_stats(r.astype(np.float64), 1e-4, k)
    for name in ("order", "selected"):
        np.testing.assert_array_equal(out[name].cpu().numpy(), want[name])
    for name in ("mean", "std", "adv"):
        np.testing.assert_allclose(out[name].cpu().numpy(), want[name], rtol=1e-5, atol=1e-6)


# 256 | 257 seeds; powers of two and their neighbours; the largest group; 16384 | 16512 rewards in all
@pytest.mark.parametrize("g,n,k", [(1, 1, 1), (3, 2, 2), (128, 128, 5), (129, 128, 4), (4, 129, 129), (2, 255, 0),
                                   (2, 256, 7), (3, 257, 8), (70, 200, 9), (2100, 8, 3), (5000, 3, 2), (2, 511, 511), (2, 512, 3), (2, 513, 2), (4, 4096, 64), (5, 4095, 3)])
@pytest.mark.parametrize("ties", [False, True])
def test_reward_sizes(d, g, n, k, ties):
    rng = np.random.default_rng(g * 10007 + n)
    r = rng.normal(size=(g, n)).astype(np.float32)
    if ties:
        r = np.round(r * 2) / 2                              # many equal values, both zeros among them
        r[r == 0] = np.where(rng.random((r == 0).sum()) < 0.5, 0.0, -0.0)
    dev, out, status = torch.from_numpy(r).cuda(), outputs(g, n, k), torch.full((1,), 99, dtype=torch.int32, device="cuda")
    d.group_reward_stats_async(dev, status, k_select=k, **out)
    assert status.item() == 0
    check(r, out, k)
    ref = outputs(g, n, k)
    d.group_reward_stats(dev, k_select=k, **ref)
    for name in ref:
        assert torch.equal(ref[name], out[name])


@pytest.mark.parametrize("g,n", [(4, 16), (3, 300), (200, 128)])
def test_reward_not_finite_writes_nothing(d, g, n):
    r = torch.rand(g, n, device="cuda")
    r[g - 1, n - 1] = float("inf")
    out, status = outputs(g, n, 2), torch.zeros(1, dtype=torch.int32, device="cuda")
    before = {k: v.clone() for k, v in out.items()}
    d.group_reward_stats_async(r, status, k_select=2, **out)
    assert status.item() == 4
    for k, v in out.items():
        assert torch.equal(v.view(torch.int32), before[k].view(torch.int32))


def test_reward_advantages_in_place(d):
    """adv over the rewards themselves: every group is checked before any is overwritten."""
    rng = np.random.default_rng(5)
    r = rng.random((64, 16)).astype(np.float32)
    dev, out, status = torch.from_numpy(r).cuda(), outputs(64, 16, 4), torch.ones(1, dtype=torch.int32, device="cuda")
    out["adv"] = dev
    d.group_reward_stats_async(dev, status, k_select=4, **out)
    assert status.item() == 0
    check(r, out, 4)
