"""GPU parity of the filter's two kernels over ranges of tiles and of the
partition's scatter: row counts at the edges of masks, tiles and the 512 ranges,
selections, column types and counts, fanouts on both sides of the kernels'
choices, and an arena too small for the masks, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FTILE, PTILE = 8192, 4096
SIZES = [0, 1, 63, 64, 65, PTILE - 1, PTILE, PTILE + 1, FTILE - 1, FTILE, FTILE + 1, 512 * PTILE - 1, 512 * PTILE + 1,
         512 * FTILE, 512 * FTILE + 5, 5_000_011]


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def ctx(gpu):
    c = gpu.Ctx(0, 1 << 30)
    yield c
    c.close()


def check_filter(gpu, c, cols, preds):
    sel, nsel = gpu.filter(c, [dev(x) for x in cols], preds)
    c.check()
    want = oracle.filter(cols, preds)
    m = int(nsel.item())
    assert m == len(want)
    np.testing.assert_array_equal(sel[:m].cpu().numpy(), want)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("bound", [-1, 3, 500, 1000])
def test_filter(gpu, ctx, n, bound):
    rng = np.random.default_rng(n)
    cols = [rng.integers(0, 1000, n).astype(np.int32), rng.integers(-2**40, 2**40, n)]
    check_filter(gpu, ctx, cols, [(0, "<", bound), (1, "!=", 0)])


def test_filter_without_room_for_the_masks(gpu):
    c = gpu.Ctx(0, 64 << 10)
    n = 3_000_001
    check_filter(gpu, c, [np.random.default_rng(1).integers(0, 9, n).astype(np.int32)], [(0, ">", 3)])
    c.close()


def check_partition(gpu, c, key, pays, fanout, sel):
    kw = {}
    if sel is not None:
        kw = {"sel": dev(sel) if len(sel) else dev(np.zeros(1, np.int32)), "nsel": dev(np.array([len(sel)], np.int64))}
    ok, op, off = gpu.partition(c, dev(key), [dev(x) for x in pays], fanout, **kw)
    c.check()
    wk, wp, woff = oracle.partition(key, pays, fanout, sel)
    m = len(wk)
    np.testing.assert_array_equal(off.cpu().numpy(), woff)
    np.testing.assert_array_equal(ok[:m].cpu().numpy(), wk)
    for g, x in zip(op, wp):
        np.testing.assert_array_equal(g[:m].cpu().numpy(), x)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("fanout,kt,picked", [(1, np.int32, None), (8, np.int64, 0.5), (9, np.int32, 0.01), (64, np.int32, None),
                                              (65, np.int64, None), (200, np.int64, 0.5), (256, np.int32, 1.0),
                                              (257, np.int32, None)])
def test_partition(gpu, ctx, n, fanout, kt, picked):
    rng = np.random.default_rng(n + fanout)
    info = np.iinfo(kt)
    key = rng.integers(info.min, info.max, n, dtype=kt, endpoint=True)
    pays = [rng.integers(0, 2407, n).astype(np.int32), rng.integers(-2**62, 2**62, n)]
    sel = None if picked is None else np.nonzero(rng.random(n) < picked)[0].astype(np.int32)
    check_partition(gpu, ctx, key, pays, fanout, sel)


@pytest.mark.parametrize("npay", [0, 1, 15])
def test_partition_one_hot_destination_and_payload_counts(gpu, ctx, npay):
    rng = np.random.default_rng(npay)
    n = 300_007
    key = np.where(rng.random(n) < 0.95, 42, rng.integers(0, 1000, n)).astype(np.int32)
    pays = [rng.integers(-2**31, 2**31, n).astype(np.int32 if j % 3 else np.int64) for j in range(npay)]
    check_partition(gpu, ctx, key, pays, 128, None)


@pytest.mark.parametrize("n", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 18) + 63, (1 << 18) + 8191, (1 << 18) + 8192,
                               (1 << 18) + 8193, 300_001])
@pytest.mark.parametrize("bound", [-1, 500, 1000])
def test_filter_where_two_kernels_take_over(gpu, ctx, n, bound):
    rng = np.random.default_rng(n)
    check_filter(gpu, ctx, [rng.integers(0, 1000, n).astype(np.int32)], [(0, "<", bound)])
