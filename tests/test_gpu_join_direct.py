"""GPU parity of the materializing join's array over dense build keys (large
sides, unique keys): ranges on both sides of the limit at which it gives way to
the hash table, slice and tile edges, key types, keys outside the range, and
its errors, against numpy indexing.  Integers: equality, no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MIN = 1 << 21       # rows of a side below which the hash table is used
SLICE = 1 << 19
TILE = 8192


@pytest.fixture(scope="module")
def ctx(gpu):
    c = gpu.Ctx(0, 4 << 30)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def capacity(nb, load=0.5):
    need = max(int(nb / load) + 1, nb + 1, 64)
    return 1 << (need - 1).bit_length()


def tables(rng, nb, npr, span, base, bt, pt):
    """nb distinct build keys that span exactly [base, base + span), and probes around them."""
    off = np.sort(rng.choice(span, nb, replace=False)) if span < 4 * nb else np.unique(rng.integers(0, span, 2 * nb))[:nb]
    off[0], off[-1] = 0, span - 1
    bk = rng.permutation(off + base).astype(bt)
    lo, hi = max(np.iinfo(pt).min, base - span // 2), min(np.iinfo(pt).max, base + span + span // 2)
    pk = rng.integers(lo, hi, npr, endpoint=True).astype(pt)
    pk[:4] = [base, base + span - 1, np.iinfo(pt).min, np.iinfo(pt).max]  # the least value is EMPTY: matches nothing
    return bk, pk


def expect(bk, pk):
    order = np.argsort(bk, kind="stable")
    at = np.clip(np.searchsorted(bk[order].astype(np.int64), pk.astype(np.int64)), 0, len(bk) - 1)
    row = order[at]
    hit = (bk[row].astype(np.int64) == pk.astype(np.int64)) & (pk != np.iinfo(pk.dtype).min)
    prow = np.nonzero(hit)[0]
    return prow, row[prow]


def check(gpu, ctx, bk, pk, **kw):
    wp, wb = expect(bk, pk)
    bc, pc = np.arange(len(bk)) * 3 - 7, np.arange(len(pk)) * 5 + 1
    prow, brow, cols, ng = gpu.join_materialize(ctx, dev(bk), [dev(bc)] * 2, dev(pk), [dev(pc)], **kw)
    ctx.check()
    m = int(ng.item())
    assert m == len(wp)
    np.testing.assert_array_equal(prow[:m].cpu().numpy(), wp)
    np.testing.assert_array_equal(brow[:m].cpu().numpy(), wb)
    np.testing.assert_array_equal(cols[0][:m].cpu().numpy(), pc[wp])
    np.testing.assert_array_equal(cols[2][:m].cpu().numpy(), bc[wb])


@pytest.mark.parametrize("nb,npr", [(MIN - 1, MIN), (MIN, MIN - 1), (MIN, MIN), (MIN + 1, MIN + 1), (MIN + 77, 3 * TILE * 128 + 1),
                                    (5_000_011, 4_000_037)])
def test_dense_keys(gpu, ctx, nb, npr):
    rng = np.random.default_rng(nb)
    check(gpu, ctx, *tables(rng, nb, npr, nb, 1, np.int32, np.int32))


@pytest.mark.parametrize("bt,pt", [(np.int32, np.int32), (np.int32, np.int64), (np.int64, np.int32), (np.int64, np.int64)])
@pytest.mark.parametrize("extra", [-SLICE, -1, 0, 1, SLICE])
def test_around_the_range_limit(gpu, ctx, bt, pt, extra):
    rng = np.random.default_rng(extra + SLICE)
    nb = MIN + 5
    base = -2**31 + 1 if bt == np.int32 else -2**40
    if pt == np.int32:
        base = -2**31 + 1
    check(gpu, ctx, *tables(rng, nb, MIN + 3, capacity(nb) + extra, base, bt, pt))


@pytest.mark.parametrize("base", [-2**63 + 1, 2**63 - 1 - 4 * MIN, -3 * MIN])
def test_int64_bases(gpu, ctx, base):
    rng = np.random.default_rng(7)
    nb, span = MIN + 1, 3 * MIN
    bk = rng.permutation(np.sort(rng.choice(span, nb, replace=False))) + base
    pk = np.concatenate([bk[: MIN // 2], rng.integers(-2**63, 2**63 - 1, MIN, endpoint=True)])
    check(gpu, ctx, bk, rng.permutation(pk))


def test_no_probe_in_range_and_one_hot_key(gpu, ctx):
    rng = np.random.default_rng(8)
    bk = rng.permutation(np.arange(MIN, dtype=np.int32))
    check(gpu, ctx, bk, np.full(MIN, MIN + 9, np.int32))
    check(gpu, ctx, bk, np.full(MIN + 1, 12345, np.int32))


def test_errors(gpu, ctx):
    rng = np.random.default_rng(9)
    bk, pk = rng.permutation(np.arange(MIN, dtype=np.int32)), rng.integers(0, MIN, MIN).astype(np.int32)
    dup = bk.copy()
    dup[5] = dup[6]
    empty = bk.copy()
    empty[17] = -2**31
    for keys, status in ((dup, gpu.ERR_DUP_KEY), (empty, gpu.ERR_KEY)):
        gpu.join_materialize(ctx, dev(keys), [], dev(pk), [])
        with pytest.raises(gpu.PystError) as e:
            ctx.check()
        assert e.value.status == status
    _, _, _, ng = gpu.join_materialize(ctx, dev(bk), [], dev(pk), [], out_cap=1000)
    with pytest.raises(gpu.PystError) as e:
        ctx.check()
    assert e.value.status == gpu.ERR_CAPACITY and int(ng.item()) == MIN


def test_arena_without_room_for_the_moves(gpu):
    nb = MIN + 9
    c = gpu.Ctx(0, capacity(nb) * 8 + nb * 16 + (4 << 20))  # the table and the packed rows, and little else
    rng = np.random.default_rng(10)
    check(gpu, c, *tables(rng, nb, MIN, nb, 0, np.int32, np.int32))
    c.close()


@pytest.mark.parametrize("bcols", [1, 2])
def test_arenas_from_the_least_to_room_for_the_moves(gpu, bcols):
    # the least: the table and the larger of the probe's words and the packed rows, which are not
    # needed at once; then up to where the optional moves (8 + 3 bytes a row and their counts) fit
    # whole, some 256 bytes short of it, and past it
    rng = np.random.default_rng(11)
    nb = MIN + 9
    bk, pk = tables(rng, nb, MIN + 5, nb, 0, np.int32, np.int32)
    wp, wb = expect(bk, pk)
    words = -(-(8 * (-(-len(pk) // 4096) + 1)) // 256) * 256
    least = 1024 + capacity(nb) * 8 + max(words, -(-(nb * 16) // 256) * 256 if bcols > 1 else 0)
    tiles, parts = -(-len(pk) // TILE), min(512, -(-nb // TILE))
    r = lambda b: -(-b // 256) * 256  # noqa: E731
    moves = (256 + 2 * 2048 * 8 + r((parts + 2 * -(-parts // 16)) * 256 * 4) + r(8 * nb) + r(tiles * 8) + r(2 * len(pk))
             + r(tiles * TILE) + r(tiles * 1024) + r(tiles * 4))
    dbk, dpk = dev(bk), dev(pk)
    bc, pc = [dev(np.arange(nb) * 3 - 7)] * bcols, [dev(np.arange(len(pk)) * 5 + 1)]
    for more in (0, 256, 1 << 20, moves - 256, moves, moves + words - 256, moves + words, moves + (1 << 20)):
        c = gpu.Ctx(0, least + more)
        prow, brow, cols, ng = gpu.join_materialize(c, dbk, bc, dpk, pc)
        c.check()
        m = int(ng.item())
        assert m == len(wp), more
        np.testing.assert_array_equal(prow[:m].cpu().numpy(), wp)
        np.testing.assert_array_equal(brow[:m].cpu().numpy(), wb)
        np.testing.assert_array_equal(cols[-1][:m].cpu().numpy(), wb * 3 - 7)
        c.close()


PIECE = 1 << 18  # least keys of a slice


@pytest.mark.parametrize("span", [8 * PIECE - 1, 8 * PIECE, 8 * PIECE + 1, 12 * PIECE - 1, 12 * PIECE, 12 * PIECE + 1])
def test_whole_slices(gpu, ctx, span):
    rng = np.random.default_rng(span)
    nb = MIN if span >= MIN else span
    bk, pk = tables(rng, nb, MIN + 3, span, -5, np.int32, np.int64)
    pk[:40] = -5 + np.clip(np.repeat(np.arange(20) * PIECE, 2) + np.tile([-1, 0], 20), 0, None)
    check(gpu, ctx, bk, pk)


def load_for(nb, slots):
    """A load under which nb rows take that power of two of slots."""
    load = nb / (slots * 0.9)
    assert capacity(nb, load) == slots
    return load


@pytest.mark.parametrize("span", [(1 << 26) + 1, (1 << 27) - 1, 1 << 27, (1 << 27) + 1])
@pytest.mark.parametrize("bt", [np.int32, np.int64])
def test_ranges_of_larger_slices(gpu, ctx, span, bt):
    # over 256 slices of 2^18 keys: twice as many keys a slice
    rng = np.random.default_rng(span)
    nb = MIN + 7
    bk, pk = tables(rng, nb, MIN + 3, span, 11, bt, np.int32)
    check(gpu, ctx, bk, pk, max_load=load_for(nb, 1 << 27))


def test_range_beyond_32_bits(gpu):
    # keys in pairs 2^32 apart, fewer values than the table has slots: their offsets do not fit 32 bits
    import torch
    slots = 1 << 33
    budget = 16 * slots + (1 << 30)
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < budget + (8 << 30):
        pytest.skip("a table of 2^33 16-byte slots does not fit the free memory")
    rng = np.random.default_rng(12)
    low = np.sort(rng.choice(1 << 24, MIN // 2 + 1, replace=False))
    bk = rng.permutation(np.concatenate([low, low + (1 << 32)])) - 3
    pk = rng.permutation(np.concatenate([bk[:MIN // 2], bk[:MIN] + 1, [2**33, -4, 2**63 - 1, -2**63]]))
    c = gpu.Ctx(0, budget)
    check(gpu, c, bk, pk, max_load=load_for(len(bk), slots))
    c.close()
