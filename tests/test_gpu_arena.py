"""The arena under blocks that are split, freed and joined again: calls of
changing sizes on one stream leave room for one that takes most of the arena, and
calls that alternate between two streams compute what they do alone.  Integers:
equality, no tolerance."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def lookup(gpu, c, k, stream=None):
    t = gpu.join_build(c, k, stream=stream)
    return t, gpu.join_probe(c, t, k, stream=stream)


@pytest.mark.parametrize("order", ["growing", "shrinking", "mixed"])
def test_changing_sizes_leave_one_block(gpu, order):
    budget = 96 << 20
    c = gpu.Ctx(0, budget)
    rng = np.random.default_rng(3)
    sizes = np.unique(np.exp(rng.uniform(np.log(100), np.log(1_500_000), 40)).astype(int))
    sizes = {"growing": sizes, "shrinking": sizes[::-1], "mixed": rng.permutation(sizes)}[order]
    large = dev(rng.permutation(5_000_000).astype(np.int32))  # its table: 2^23 slots of 8 bytes at a load of 0.9
    for n in sizes:
        k = dev(rng.permutation(n).astype(np.int32))
        held, (rows, vals, ng) = lookup(gpu, c, k)  # in between, blocks of other calls are taken and freed
        gk, gs, gn = gpu.groupby_sum(c, k, k, sort_by_key=True)
        other = gpu.join_build(c, k[: n // 2 + 1].contiguous())
        held.destroy()
        gpu.partition(c, k, [k], 7)
        other.destroy()
        c.check()
        assert int(ng.item()) == n and int(gn.item()) == n
        np.testing.assert_array_equal(vals[:n].cpu().numpy(), np.arange(n))
        np.testing.assert_array_equal(gk[:n].cpu().numpy(), np.arange(n))
        assert c.used == 0
        t = gpu.join_build(c, large, max_load=0.9)
        c.check()
        t.destroy()
    c.close()


def test_freed_blocks_are_one_again_without_a_wait(gpu):
    # no check, no destroy and no other call that waits: the same stream's next call finds the whole
    c = gpu.Ctx(0, 96 << 20)
    rng = np.random.default_rng(4)
    large = dev(rng.integers(0, 1 << 40, 1_500_000))
    small = [dev(rng.integers(0, 1 << 40, n)) for n in (70, 900_000, 3_000, 400_000, 11)]
    want = [oracle.groupby_sum(k.cpu().numpy(), k.cpu().numpy(), None) for k in small + [large]]
    got = []
    for _ in range(5):
        got = [gpu.groupby_sum(c, k, k, sort_by_key=True) for k in small + [large]]
    c.check()
    for (gk, gs, gn), (wk, ws) in zip(got, want):
        m = int(gn.item())
        assert m == len(wk)
        np.testing.assert_array_equal(gk[:m].cpu().numpy(), wk)
        np.testing.assert_array_equal(gs[:m].cpu().numpy(), ws)
    c.close()


def test_two_streams_over_the_same_blocks(gpu):
    import torch
    c = gpu.Ctx(0, 160 << 20)  # too little for both streams' calls at their largest
    rng = np.random.default_rng(5)
    streams = [torch.cuda.Stream() for _ in range(2)]
    keys = [rng.integers(-2**40, 2**40, n) for n in (1_200_000, 50_000, 700_001, 3_000, 1_100_000, 257)]
    want = [oracle.groupby_sum(k, k, None) for k in keys]
    perms = [rng.permutation(n).astype(np.int32) for n in (900_000, 2_000, 300_001)]
    dk, dp = [dev(k) for k in keys], [dev(p) for p in perms]
    torch.cuda.synchronize()
    groups, finds = [], []
    for turn in range(18):
        s = streams[turn % 2 if turn % 5 else 0]
        with torch.cuda.stream(s):
            i = turn % len(keys)
            groups.append((i, gpu.groupby_sum(c, dk[i], dk[i], sort_by_key=True, stream=s)))
            j = turn % len(perms)
            t, found = lookup(gpu, c, dp[j], stream=s)
            finds.append((j, found))
            if turn % 3:
                t.destroy(stream=s)  # the other stream's blocks stay where they are
            else:
                groups.append((i, gpu.groupby_sum(c, dk[i], dk[i], sort_by_key=True, stream=s)))
                t.destroy(stream=s)
    for s in streams:
        c.check(s)
    torch.cuda.synchronize()
    for i, (gk, gs, gn) in groups:
        m = int(gn.item())
        assert m == len(want[i][0])
        np.testing.assert_array_equal(gk[:m].cpu().numpy(), want[i][0])
        np.testing.assert_array_equal(gs[:m].cpu().numpy(), want[i][1])
    for j, (rows, vals, ng) in finds:
        n = len(perms[j])
        assert int(ng.item()) == n
        np.testing.assert_array_equal(rows[:n].cpu().numpy(), np.arange(n))
        np.testing.assert_array_equal(vals[:n].cpu().numpy(), np.arange(n))
    assert c.used == 0
    c.close()
