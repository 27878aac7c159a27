"""GPU parity of the group-by's key-range plans (LDS arrays over a small range,
ranged buckets in key order) and of the hash buckets and table they give way
to, at the edges where the choice changes, against the oracle.  Sums are exact
integers: equality, no tolerance."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SMALL, RANGED = 8192, 1 << 25


@pytest.fixture(scope="module")
def ctx(gpu):
    c = gpu.Ctx(0, 4 << 30)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def keys_over(rng, n, span, base, dtype):
    """n keys that span exactly [base, base + span)."""
    k = rng.integers(0, span, n)
    k[0], k[-1] = 0, span - 1
    return (k + base).astype(dtype)


def check(gpu, ctx, k, v, sel=None, **kw):
    if sel is not None:
        kw.update(sel=dev(sel) if len(sel) else dev(np.zeros(1, np.int32)), nsel=dev(np.array([len(sel)], np.int64)))
    gk, gs, ng = gpu.groupby_sum(ctx, dev(k), dev(v), sort_by_key=True, **kw)
    ctx.check()
    m = int(ng.item())
    wk, ws = oracle.groupby_sum(k, v, sel)
    assert m == len(wk)
    np.testing.assert_array_equal(gk[:m].cpu().numpy(), wk)
    np.testing.assert_array_equal(gs[:m].cpu().numpy(), ws)


@pytest.mark.parametrize("kt,vt", [(np.int32, np.int32), (np.int32, np.int64), (np.int64, np.int64),
                                   (np.int64, np.int32)])
@pytest.mark.parametrize("span,base", [(1, -5), (2, 0), (63, 7), (512, -1), (SMALL - 1, -100), (SMALL, -2**31 + 1),
                                       (SMALL + 1, -SMALL), (100_000, -2**31 + 1), (RANGED - 1, 3), (RANGED, -RANGED // 2),
                                       (RANGED + 1, 0)])
def test_key_ranges(gpu, ctx, kt, vt, span, base):
    rng = np.random.default_rng(span)
    n = (1 << 20) + 17
    k = keys_over(rng, n, span, base, kt)
    info = np.iinfo(vt)
    check(gpu, ctx, k, rng.integers(info.min, info.max, n, dtype=vt, endpoint=True))


@pytest.mark.parametrize("vt", [np.int32, np.int64])
@pytest.mark.parametrize("span", [3000, 1_000_000])
@pytest.mark.parametrize("picked", [0, 1, 100_003])
def test_selections(gpu, ctx, vt, span, picked):
    rng = np.random.default_rng(picked + span)
    n = 1 << 20
    k = keys_over(rng, n, span, 11, np.int32)
    sel = np.sort(rng.choice(n, picked, replace=False)).astype(np.int32)
    check(gpu, ctx, k, rng.integers(-1000, 1000, n).astype(vt), sel)


@pytest.mark.parametrize("vt", [np.int32, np.int64])
def test_crowded_keys_take_hash_buckets(gpu, ctx, vt):
    # half of the rows in one value, the rest in a far narrower range than the whole
    rng = np.random.default_rng(5)
    n = 1_500_000
    k = np.where(rng.random(n) < 0.5, 77, rng.integers(0, 40_000, n)).astype(np.int32)
    k[1] = 20_000_000
    check(gpu, ctx, k, rng.integers(-1000, 1000, n).astype(vt))


def test_widest_int64_range_and_sorted_input(gpu, ctx):
    rng = np.random.default_rng(6)
    n = 1 << 20
    k = rng.integers(-2**63 + 1, 2**63 - 1, n, endpoint=True)
    k[:2] = [-2**63 + 1, 2**63 - 1]
    check(gpu, ctx, k, rng.integers(-2**62, 2**62, n))
    check(gpu, ctx, np.sort(keys_over(rng, n, 900_000, -450_000, np.int64)), rng.integers(-2**62, 2**62, n))


@pytest.mark.parametrize("span", [900, 5_000_000])
def test_over_max_groups_keeps_the_count(gpu, ctx, span):
    n = 1 << 20
    rng = np.random.default_rng(span)
    k, v = keys_over(rng, n, span, 0, np.int32), np.ones(n, np.int32)
    need = len(np.unique(k))
    gk, gs, ng = gpu.groupby_sum(ctx, dev(k), dev(v), max_groups=need - 1)
    with pytest.raises(gpu.PystError) as e:
        ctx.check()
    assert e.value.status == gpu.ERR_CAPACITY and int(ng.item()) == need


@pytest.mark.parametrize("kt,span", [(np.int32, 2500), (np.int32, 3_000_000), (np.int64, 1 << 40)])
@pytest.mark.parametrize("budget", [4 << 30, 1200 << 20])
def test_unbounded_groups(gpu, kt, span, budget):
    # more rows than hash buckets take (2^24) and no bound on the groups: ranges where the arena
    # has room for the moves beside the table in HBM, else the table
    c = gpu.Ctx(0, budget)
    rng = np.random.default_rng(9)
    n = (1 << 24) + 5
    k, v = keys_over(rng, n, span, -9, kt), rng.integers(-2**31, 2**31, n).astype(np.int32)
    gk, gs, ng = gpu.groupby_sum(c, dev(k), dev(v))
    c.check()
    m = int(ng.item())
    gk, gs = gk[:m].cpu().numpy(), gs[:m].cpu().numpy()
    o = np.argsort(gk)
    wk, ws = oracle.groupby_sum(k, v)
    np.testing.assert_array_equal(gk[o], wk)
    np.testing.assert_array_equal(gs[o], ws)
    c.close()


@pytest.mark.parametrize("kt", [np.int32, np.int64])
@pytest.mark.parametrize("n", [1, 1023, 4097, 200_001, (1 << 20) + 1, 3_000_000])
@pytest.mark.parametrize("groups", [1, 5, 1400, 4096, 30_000])
def test_few_keys_over_a_wide_range(gpu, ctx, kt, n, groups):
    # below 2^20 rows the table behind per-block LDS tables, above it the plan's choice
    rng = np.random.default_rng(n + groups)
    info = np.iinfo(kt)
    pool = rng.integers(info.min + 1, info.max, groups, dtype=kt, endpoint=True)
    pool[0], pool[-1] = info.min + 1, info.max
    k = pool[rng.integers(0, groups, n)]
    v = rng.integers(-2**62, 2**62, n)
    check(gpu, ctx, k, v)
    if n > 2:
        check(gpu, ctx, k, v, np.arange(1, n, 2, dtype=np.int32))


@pytest.mark.parametrize("unbounded", [False, True])
def test_sample_promises_too_few_keys(gpu, ctx, unbounded):
    # 19 rows of 20 in 100 keys, the rest all different: the sample finds under 1500 keys, the
    # table of 2^16 slots runs full, and the rows go to hash buckets (or the table in HBM)
    rng = np.random.default_rng(3)
    n = (1 << 24) + 7 if unbounded else 4_000_000
    k = np.where(rng.random(n) < 0.95, rng.integers(0, 100, n) << 50, rng.integers(-2**62, 2**62, n))
    check(gpu, ctx, k, rng.integers(-2**62, 2**62, n), max_groups=0 if unbounded else n)


@pytest.mark.parametrize("n", [1 << 20, (1 << 22) + 12_345])
@pytest.mark.parametrize("span", [1 << 14, 1_000_001, (1 << 24) - 1, 1 << 24, (1 << 24) + 1])
@pytest.mark.parametrize("picked", [None, 0, 1, 16_385, 900_001])
def test_one_move_of_int32_pairs(gpu, ctx, n, span, picked):
    # spans of 2^24 values are moved once, wider ones twice; sums that cancel
    # stay groups; the last tiles of the blocks' ranges are short
    rng = np.random.default_rng(span + n)
    k = keys_over(rng, n, span, -(span // 2), np.int32)
    v = rng.integers(-2**31, 2**31, n).astype(np.int32)
    v[k % 3 == 0] = 0
    sel = None if picked is None else np.sort(rng.choice(n, picked, replace=False)).astype(np.int32)
    check(gpu, ctx, k, v, sel)


@pytest.mark.parametrize("share", [0.004, 0.01, 0.012, 0.1])
def test_crowded_buckets_of_one_move(gpu, ctx, share):
    # a run of 4096 neighbouring keys with that share of the rows: the buckets of
    # one move, or those of two, or neither take them
    rng = np.random.default_rng(7)
    n, span = 3_000_017, 1 << 22
    k = keys_over(rng, n, span, 0, np.int32)
    many = rng.random(n) < share
    k[many] = rng.integers(1 << 20, (1 << 20) + 4096, int(many.sum()))
    check(gpu, ctx, k, rng.integers(-2**31, 2**31, n).astype(np.int32))


@pytest.mark.parametrize("kt", [np.int32, np.int64])
@pytest.mark.parametrize("skip", [0, 1, 2, 3])
@pytest.mark.parametrize("extra", [0, 1, 2, 3])
def test_key_columns_off_16_bytes(gpu, ctx, kt, skip, extra):
    # the range is read in 16-byte words where the column allows it; the least
    # and greatest keys are the first and last rows
    rng = np.random.default_rng(skip)
    n = (1 << 20) + extra
    k = keys_over(rng, n, 50_000, -7, kt)
    v = rng.integers(-100, 100, n).astype(np.int32)
    d = dev(np.concatenate([np.full(skip, 10**9, kt), k]))[skip:]
    gk, gs, ng = gpu.groupby_sum(ctx, d, dev(v), sort_by_key=True)
    ctx.check()
    wk, ws = oracle.groupby_sum(k, v)
    m = int(ng.item())
    np.testing.assert_array_equal(gk[:m].cpu().numpy(), wk)
    np.testing.assert_array_equal(gs[:m].cpu().numpy(), ws)


def test_few_table_full_while_blocks_still_start(gpu):
    # two streams share the chip, so blocks start after others have found the table full
    import torch
    rng = np.random.default_rng(41)
    n = 4_000_000
    k = np.where(rng.random(n) < 0.95, rng.integers(0, 100, n) << 50, rng.integers(-2**62, 2**62, n))
    v = rng.integers(-2**62, 2**62, n)
    wk, ws = oracle.groupby_sum(k, v)
    dk, dv = dev(k), dev(v)
    ctxs = [gpu.Ctx(0, 1 << 30) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    got = []
    for _ in range(3):
        for c, s in zip(ctxs, streams):
            with torch.cuda.stream(s):
                got.append(gpu.groupby_sum(c, dk, dv, max_groups=n, sort_by_key=True, stream=s))
    for c, s in zip(ctxs, streams):
        c.check(s)
    torch.cuda.synchronize()
    for gk, gs, ng in got:
        m = int(ng.item())
        assert m == len(wk)
        np.testing.assert_array_equal(gk[:m].cpu().numpy(), wk)
        np.testing.assert_array_equal(gs[:m].cpu().numpy(), ws)
    for c in ctxs:
        c.close()


def rounded(b):
    return (b + 255) // 256 * 256


def test_table_comes_before_what_a_plan_takes(gpu):
    # arenas that hold the table in HBM and its compaction words, and beside them any first part
    # of the memory that a plan takes where there is room: the moves' two buffers, the plan, the
    # few-keys table; each leaves 256 bytes less than the words would need after it
    rng = np.random.default_rng(13)
    n = (1 << 24) + 5
    k = rng.integers(0, 100_000, n) * 1_000_003 - 2**40
    v = rng.integers(-2**31, 2**31, n).astype(np.int32)
    wk, ws = oracle.groupby_sum(k, v)
    dk, dv = dev(k), dev(v)
    slots = 1 << 25  # n rows at a load of 0.9
    table, words = 1024 + 16 * slots, rounded(8 * (slots // 2048 + 1))
    parts, buckets = 64 * 512, 4096 * 8
    counts = rounded(4 * (512 * 4096 + 2 * (parts + 1 + buckets + 1)))
    plan = rounded(256 + 8 * 4096 + 16 * 2048 + 8 * 16384)
    few = rounded(1024 + 16 * 65536 + 8 * (65536 // 2048 + 1))
    optional = [rounded(16 * n), rounded(counts + 16 * n), plan, few]
    for held in range(len(optional) + 1):
        c = gpu.Ctx(0, table + words + max(0, sum(optional[:held]) - 256))
        gk, gs, ng = gpu.groupby_sum(c, dk, dv, max_load=0.9)
        c.check()
        m = int(ng.item())
        assert m == len(wk), held
        o = np.argsort(gk[:m].cpu().numpy())
        np.testing.assert_array_equal(gk[:m].cpu().numpy()[o], wk)
        np.testing.assert_array_equal(gs[:m].cpu().numpy()[o], ws)
        c.close()


@pytest.mark.parametrize("kt,vt", [(np.int32, np.int32), (np.int64, np.int64)])
@pytest.mark.parametrize("span", [SMALL + 1, 1 << 31])
@pytest.mark.parametrize("picked", [0, 1, 1024, 1025, 8192, 8193, 32768, 32769])
def test_few_selected_rows(gpu, ctx, kt, vt, span, picked):
    # up to these numbers of rows the table takes them, whatever their keys
    rng = np.random.default_rng(picked)
    n = 1 << 20
    k = keys_over(rng, n, span, -2**31, kt)
    info = np.iinfo(vt)
    v = rng.integers(info.min, info.max, n, dtype=vt, endpoint=True)
    check(gpu, ctx, k, v, np.sort(rng.choice(n, picked, replace=False)).astype(np.int32))
    check(gpu, ctx, np.full(n, k[1]), v, np.sort(rng.choice(n, picked, replace=False)).astype(np.int32))


def time_groupby(gpu, ctx, *args, **kw):
    import torch
    best = []
    for _ in range(7):
        gpu.groupby_sum(ctx, *args, max_groups=1 << 20, **kw)
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            gpu.groupby_sum(ctx, *args, max_groups=1 << 20, **kw)
        b.record()
        b.synchronize()
        best.append(a.elapsed_time(b))
    return min(best)


def test_few_selected_rows_cost_what_few_rows_do(gpu, ctx):
    # 1000 of 8M rows, random 64-bit keys, against a column of 1000 rows.  By hash buckets the first takes
    # over ten times as long; the limit lies between that and the launches that choose.
    rng = np.random.default_rng(8)
    n = 8_000_000
    k, v = dev(rng.integers(0, 1 << 40, n)), dev(rng.integers(0, 99, n))
    sel = np.sort(rng.choice(n, 1000, replace=False)).astype(np.int32)
    few = time_groupby(gpu, ctx, k, v, sel=dev(sel), nsel=dev(np.array([1000], np.int64)))
    column = time_groupby(gpu, ctx, k[:1000].contiguous(), v[:1000].contiguous())
    ctx.check()
    assert few < 5 * column, (few, column)


@pytest.mark.parametrize("kt", [np.int32, np.int64])
@pytest.mark.parametrize("picked", [(1 << 19) - 1, 1 << 19, 700_001])
@pytest.mark.parametrize("case", ["narrow", "outlier read first", "outlier between", "wide", "few and wide"])
def test_large_selections_are_judged_by_some_of_their_keys(gpu, ctx, kt, picked, case):
    # from 2^19 selected rows on, 256 of them (the first among them) may already span more than any range mode takes
    rng = np.random.default_rng(picked)
    n = (1 << 20) + 3
    k = keys_over(rng, n, 60_000, -30_000, kt)
    sel = np.sort(rng.choice(n, picked, replace=False)).astype(np.int32)
    if case == "outlier read first":
        k[sel[0]] = 2**31 - 1
    elif case == "outlier between":
        k[sel[1]] = 2**31 - 1
    elif case == "wide":
        k = keys_over(rng, n, 1 << 32, -2**31, kt)
    elif case == "few and wide":
        k = rng.choice(keys_over(rng, 9, 1 << 32, -2**31, kt), n)
    check(gpu, ctx, k, rng.integers(-1000, 1000, n), sel)


@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("keys", [9, 1 << 40])
def test_empty_key_of_a_large_selection(gpu, ctx, at, keys):
    rng = np.random.default_rng(at)
    n = 1 << 20
    k = rng.choice(rng.integers(-2**62, 2**62, 9), n) if keys == 9 else rng.integers(0, keys, n)
    sel = np.arange(0, n, 2, dtype=np.int32)
    k[sel[at]] = np.iinfo(np.int64).min
    gpu.groupby_sum(ctx, dev(k), dev(k), sel=dev(sel), nsel=dev(np.array([len(sel)], np.int64)))
    with pytest.raises(gpu.PystError) as e:
        ctx.check()
    assert e.value.status == gpu.ERR_KEY


@pytest.mark.parametrize("picked", [0, 1, 1000, 1023, 1024, 2047, 2048, 20_001, 300_000])
def test_tables_that_use_a_part_of_their_slots(gpu, ctx, picked):
    # the compaction's tiles (2048 slots) end with the slots in use: 64 at least, twice the selected rows
    rng = np.random.default_rng(picked)
    n = 300_000
    k = rng.integers(-2**62, 2**62, n)
    check(gpu, ctx, k, rng.integers(-9, 9, n), np.sort(rng.choice(n, picked, replace=False)).astype(np.int32))


@pytest.mark.parametrize("n", [1, 127, 128, 129, 1023, 1025, 16_383, 16_384, 16_385, 131_071, 131_073, 262_143, 524_289])
@pytest.mark.parametrize("groups", [1, 1 << 40])
def test_blocks_of_few_rows(gpu, ctx, n, groups):
    # units of 128 rows while a block has fewer than 1024, units of 1024 from there
    rng = np.random.default_rng(n)
    k = rng.integers(0, groups, n)
    check(gpu, ctx, k, rng.integers(-2**62, 2**62, n))
    sel = np.sort(rng.choice(n, n // 3 + 1, replace=False)).astype(np.int32)
    check(gpu, ctx, k, rng.integers(-2**62, 2**62, n), sel)
