"""GPU parity of the group-by's ordered output where the groups have to be
sorted (the hash table in HBM): pair counts around the one-block sort's limit
and the tile size, and key ranges of every number of passes, against the
oracle.  Exact integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SMALL, TILE = 8192, 4096


@pytest.fixture(scope="module")
def ctx(gpu):
    c = gpu.Ctx(0, 2 << 30)
    c.groupby_hash_only(True)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def distinct(rng, n, bits, dtype):
    """n distinct keys that span exactly 2^bits values (or all of the type but its EMPTY value)."""
    info = np.iinfo(dtype)
    lo = info.min + 1 if bits >= info.bits else int(rng.integers(info.min + 1, info.max - 2**bits + 2))
    hi = info.max if bits >= info.bits else lo + 2**bits - 1
    if hi - lo < 4 * n:
        k = lo + rng.permutation(hi - lo + 1)[:n]
    else:
        k = np.unique(rng.integers(lo, hi, 2 * n, dtype=np.int64, endpoint=True))
        k = rng.permutation(k)[:n]
    k[0], k[-1] = lo, hi
    return np.unique(k).astype(dtype)


def check(gpu, ctx, k, v, **kw):
    gk, gs, ng = gpu.groupby_sum(ctx, dev(k), dev(v), sort_by_key=True, **kw)
    ctx.check()
    m = int(ng.item())
    wk, ws = oracle.groupby_sum(k, v)
    assert m == len(wk)
    np.testing.assert_array_equal(gk[:m].cpu().numpy(), wk)
    np.testing.assert_array_equal(gs[:m].cpu().numpy(), ws)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, TILE, SMALL - 1, SMALL, SMALL + 1, 3 * TILE - 1,
                               3 * TILE, 3 * TILE + 1, 100_003, 1_500_000])
@pytest.mark.parametrize("bits,dtype", [(24, np.int32), (33, np.int64), (64, np.int64)])
def test_counts(gpu, ctx, n, bits, dtype):
    rng = np.random.default_rng(n)
    k = rng.permutation(distinct(rng, n, bits, dtype))
    check(gpu, ctx, k, rng.integers(-2**62, 2**62, len(k)))


@pytest.mark.parametrize("n", [5000, 40_000])
@pytest.mark.parametrize("bits,dtype", [(16, np.int32), (17, np.int32), (32, np.int32), (8, np.int64), (16, np.int64),
                                        (17, np.int64), (32, np.int64), (40, np.int64), (48, np.int64), (49, np.int64),
                                        (63, np.int64)])
def test_key_spans(gpu, ctx, n, bits, dtype):
    rng = np.random.default_rng(n + bits)
    k = distinct(rng, min(n, 2**bits), bits, dtype)
    for order in (k, k[::-1], rng.permutation(k)):
        check(gpu, ctx, order, rng.integers(-2**62, 2**62, len(k)))


def test_few_groups_in_a_large_output(gpu, ctx):
    rng = np.random.default_rng(1)
    for groups in (3, 20_000):
        k = rng.integers(0, groups, 700_000) * (1 << 33) - (1 << 60)
        check(gpu, ctx, k, rng.integers(-2**62, 2**62, len(k)))


@pytest.mark.parametrize("n,max_groups", [(50, 10_000), (50, 3_000_000), (9_000, 20_000)])
def test_output_larger_than_the_rows(gpu, n, max_groups):
    # the arena holds what a sort of eight byte passes over max_groups pairs takes beside the table:
    # the pairs again, and 256 counts and their sums per 4096 of them
    rng = np.random.default_rng(n)
    slots = 1 << (2 * n).bit_length()
    table = 1024 + 16 * slots
    tiles = (max_groups + TILE - 1) // TILE
    counts = (2 * tiles * 256 * 4 + 256 + 255) // 256 * 256 + 8 * (tiles * 256 // 2048 + 2)
    c = gpu.Ctx(0, sum((b + 255) // 256 * 256 for b in (table, 16 * max_groups, counts)))
    k = rng.permutation(distinct(rng, n, 40, np.int64))
    check(gpu, c, k, rng.integers(-9, 9, len(k)), max_groups=max_groups)
    c.close()
