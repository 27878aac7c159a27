"""GPU parity of probes of unique-key hash tables beyond the L2 (taken slice by
slice) against numpy: both slot widths, key and payload types, selections on
either side, row counts at the edges of tiles and ranges, and the errors and the
short arena that keep the other path.  Integers: equality, no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = 1 << 21  # probe rows from which a large table is probed by slices
TILE = 8192


@pytest.fixture(scope="module")
def ctx(gpu):
    c = gpu.Ctx(0, 2 << 30)
    yield c
    c.close()


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def sel_kw(sel):
    if sel is None:
        return {}
    return {"sel": dev(sel if len(sel) else np.zeros(1, np.int32)), "nsel": dev(np.array([len(sel)], np.int64))}


def expect(bk, pay, pk, bsel, psel):
    rows_b = np.arange(len(bk)) if bsel is None else bsel
    rows_p = np.arange(len(pk)) if psel is None else psel
    keys = bk[rows_b].astype(np.int64)
    order = np.argsort(keys, kind="stable")
    keys, rows_b = keys[order], rows_b[order]
    p = pk[rows_p].astype(np.int64)
    at = np.clip(np.searchsorted(keys, p), 0, max(len(keys) - 1, 0))
    hit = (keys[at] == p if len(keys) else np.zeros(len(p), bool)) & (pk[rows_p] != np.iinfo(pk.dtype).min)
    b = rows_b[at[hit]] if len(keys) else np.zeros(0, np.int64)
    return rows_p[hit], b if pay is None else pay[b].astype(np.int64)


def check(gpu, ctx, bk, pay, pk, bsel=None, psel=None):
    t = gpu.join_build(ctx, dev(bk), None if pay is None else dev(pay), **sel_kw(bsel))
    rows, vals, ng = gpu.join_probe(ctx, t, dev(pk), **sel_kw(psel))
    ctx.check()
    m = int(ng.item())
    wr, wv = expect(bk, pay, pk, bsel, psel)
    assert m == len(wr)
    np.testing.assert_array_equal(rows[:m].cpu().numpy(), wr)
    np.testing.assert_array_equal(vals[:m].cpu().numpy(), wv)
    t.destroy()


def sides(rng, nb, npr, bt, pt, wide_range):
    lo, hi = (np.iinfo(bt).min + 1, np.iinfo(bt).max) if wide_range else (0, 4 * nb)
    bk = np.unique(rng.integers(lo, hi, 2 * nb, dtype=np.int64, endpoint=True))
    bk = rng.permutation(bk)[:nb].astype(bt)
    info = np.iinfo(pt)
    hits = bk[rng.integers(0, nb, npr)].astype(np.int64)
    miss = rng.integers(info.min, info.max, npr, dtype=np.int64, endpoint=True)
    pk = np.clip(np.where(rng.random(npr) < 0.5, hits, miss), info.min, info.max).astype(pt)
    pk[:3] = [info.min, info.max, info.min + 1]
    return bk, pk


@pytest.mark.parametrize("bt,vt,pt", [(np.int32, np.int32, np.int32), (np.int32, None, np.int64), (np.int32, np.int64, np.int32),
                                      (np.int64, np.int64, np.int64), (np.int64, np.int32, np.int32), (np.int64, None, np.int64)])
@pytest.mark.parametrize("wide_range", [False, True])
def test_types(gpu, ctx, bt, vt, pt, wide_range):
    rng = np.random.default_rng(1)
    nb = 1_200_003
    bk, pk = sides(rng, nb, ROWS + 12_345, bt, pt, wide_range)
    pay = None if vt is None else rng.integers(np.iinfo(vt).min, np.iinfo(vt).max, nb, dtype=vt, endpoint=True)
    if pay is not None:
        pay[:100] = -1
    check(gpu, ctx, bk, pay, pk)


@pytest.mark.parametrize("npr", [ROWS - 1, ROWS, ROWS + 1, 512 * TILE - 1, 512 * TILE + 1])
@pytest.mark.parametrize("wide", [False, True])
def test_probe_counts(gpu, ctx, npr, wide):
    rng = np.random.default_rng(npr)
    bk, pk = sides(rng, 700_001, npr, np.int64 if wide else np.int32, np.int64 if wide else np.int32, True)
    check(gpu, ctx, bk, rng.integers(-2**31, 2**31, len(bk)).astype(np.int32), pk)


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("built,probed", [(0, 1.0), (5, 0.3), (300_000, 0.0), (None, 0.5)])
def test_selections(gpu, ctx, wide, built, probed):
    # the table's size follows the rows selected, on the device
    rng = np.random.default_rng(17)
    kt = np.int64 if wide else np.int32
    bk, pk = sides(rng, 1_100_000, ROWS + 77, kt, kt, False)
    bsel = None if built is None else np.sort(rng.choice(len(bk), built, replace=False)).astype(np.int32)
    psel = np.nonzero(rng.random(len(pk)) < probed)[0].astype(np.int32)
    check(gpu, ctx, bk, rng.integers(-2**31, 2**31, len(bk)).astype(np.int32), pk, bsel, psel)


def test_hot_key_and_capacity(gpu, ctx):
    rng = np.random.default_rng(3)
    bk = rng.permutation(np.arange(1_300_000, dtype=np.int64) << 20)
    pk = np.full(ROWS + 5, bk[77])
    check(gpu, ctx, bk, rng.integers(-9, 9, len(bk)), pk)
    t = gpu.join_build(ctx, dev(bk))
    rows, vals, ng = gpu.join_probe(ctx, t, dev(pk), out_cap=1000)
    with pytest.raises(gpu.PystError) as e:
        ctx.check()
    assert e.value.status == gpu.ERR_CAPACITY and int(ng.item()) == len(pk)
    np.testing.assert_array_equal(rows.cpu().numpy(), np.arange(1000))
    assert (vals.cpu().numpy() == 77).all()
    t.destroy()


def test_duplicate_keys_and_short_arena_keep_the_other_path(gpu):
    rng = np.random.default_rng(4)
    bk, pk = sides(rng, 1_100_000, ROWS, np.int32, np.int32, True)
    c = gpu.Ctx(0, 40 << 20)  # the 32 MiB table and no room for the slices
    check(gpu, c, bk, None, pk)
    c.close()
    c = gpu.Ctx(0, 1 << 30)
    dup = np.concatenate([bk, bk[:10]])
    t = gpu.join_build(c, dev(dup), unique_keys=False)
    rows, vals, ng = gpu.join_probe(c, t, dev(pk), out_cap=2 * len(pk))
    c.check()
    wr, _ = expect(bk, None, pk, None, None)
    extra = np.isin(pk, bk[:10]).sum()
    assert int(ng.item()) == len(wr) + extra
    t.destroy()
    c.close()


def fill_arena(gpu, c):
    """Writes the word 2^31 (an EMPTY slot) all over a context's arena, and gives it back."""
    t = gpu.join_build(c, dev(np.arange(3, dtype=np.int32)), max_load=3 / (c.budget // 2 // 8 - 2))
    t.destroy()
    c.check()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("build_sel", [False, True])
def test_empty_selection_first_in_a_used_arena(gpu, wide, build_sel):
    # no row moves, so nothing but the clearing of the scratch says so to the later kernels
    rng = np.random.default_rng(29)
    kt = np.int64 if wide else np.int32
    bk, pk = sides(rng, 1_100_000, ROWS + 77, kt, kt, False)
    pay = rng.integers(-2**31, 2**31, len(bk)).astype(np.int32)
    bsel = np.arange(1, len(bk), dtype=np.int32) if build_sel else None
    c = gpu.Ctx(0, 512 << 20)
    fill_arena(gpu, c)
    check(gpu, c, bk, pay, pk, bsel, np.zeros(0, np.int32))
    check(gpu, c, bk, pay, pk, bsel, np.array([len(pk) - 1], np.int32))
    check(gpu, c, bk, pay, pk, bsel, np.zeros(0, np.int32))
    c.close()


@pytest.mark.parametrize("wide,slots", [(False, 1 << 26), (False, 1 << 27), (True, 1 << 25), (True, 1 << 26)])
def test_slices_of_more_than_the_least_slots(gpu, ctx, wide, slots):
    # from 2^27 slots of 8 bytes and 2^26 of 16, 256 slices take more than 2 MiB each
    rng = np.random.default_rng(slots)
    kt = np.int64 if wide else np.int32
    bk, pk = sides(rng, 1_100_000, ROWS + 5, kt, kt, True)
    t = gpu.join_build(ctx, dev(bk), max_load=len(bk) / (slots * 0.9))
    assert t.info()[0] == slots
    rows, vals, ng = gpu.join_probe(ctx, t, dev(pk))
    ctx.check()
    m = int(ng.item())
    wr, wv = expect(bk, None, pk, None, None)
    assert m == len(wr)
    np.testing.assert_array_equal(rows[:m].cpu().numpy(), wr)
    np.testing.assert_array_equal(vals[:m].cpu().numpy(), wv)
    t.destroy()


LONG = 1 << 22  # rows of a column of which a small part is probed by slices, whatever the table


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("npr", [LONG - 1, LONG])
@pytest.mark.parametrize("built,probed", [(5, LONG // 4 - 2), (5, LONG // 4), (0, 0), (70_000, 1), (70_000, None),
                                          (1_099_999, LONG // 4 + 1), (1_099_999, 1000)])
def test_tables_built_from_a_selection(gpu, ctx, wide, npr, built, probed):
    # the device chooses by the slots the table uses and the rows probed
    rng = np.random.default_rng(npr + built)
    kt = np.int64 if wide else np.int32
    bk, pk = sides(rng, 1_100_000, npr, kt, kt, False)
    bsel = np.sort(rng.choice(len(bk), built, replace=False)).astype(np.int32)
    psel = None if probed is None else np.sort(rng.choice(npr, probed, replace=False)).astype(np.int32)
    check(gpu, ctx, bk, rng.integers(-2**31, 2**31, len(bk)).astype(np.int32), pk, bsel, psel)


@pytest.mark.parametrize("wide", [False, True])
def test_few_built_rows_cost_what_a_small_table_does(gpu, ctx, wide):
    # all of 2^23 rows probed in a table of five rows: selected from a large column, or a column of five.
    # By slices the first takes three (two) times as long as the second; the limit lies between that and one.
    import torch
    rng = np.random.default_rng(7)
    kt = np.int64 if wide else np.int32
    bk = rng.permutation(4_000_000).astype(kt)
    pk = dev(rng.integers(0, 4_000_000, 1 << 23).astype(kt))
    tables = [gpu.join_build(ctx, dev(bk), **sel_kw(np.arange(5, dtype=np.int32))), gpu.join_build(ctx, dev(bk[:5]))]
    times = [[], []]
    for _ in range(7):
        for t, out in zip(tables, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            gpu.join_probe(ctx, t, pk)
            a.record()
            for _ in range(10):
                gpu.join_probe(ctx, t, pk)
            b.record()
            b.synchronize()
            out.append(a.elapsed_time(b))
    ctx.check()
    assert min(times[0]) < 1.6 * min(times[1])
    for t in tables:
        t.destroy()
