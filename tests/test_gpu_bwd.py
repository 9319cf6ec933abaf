"""GPU parity of dmt_tower_lookup_bwd_update against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from harness import RTOL, DeviceWorkload, assert_close, to_f64

pytestmark = pytest.mark.gpu


def run_bwd(dw, idx, off, grad, lr, eps, debug=True):
    dmt, w = dw.dmt, dw.w
    nnz = len(idx)
    d_idx, d_off = torch.from_numpy(idx).cuda(), torch.from_numpy(off).cuda()
    d_grad = torch.from_numpy(grad).cuda()
    ws = torch.empty(max(dmt.dmt_bwd_workspace_bytes(dw.plan, w.batch, nnz), 256) // 8 + 32,
                     dtype=torch.int64, device="cuda")
    ws.fill_(-1)                         # stale scratch must not matter
    dbg = None
    if debug:
        dbg = dict(sorted_keys=torch.full((nnz,), -7, dtype=torch.int64, device="cuda"),
                   sorted_bag=torch.full((nnz,), -7, dtype=torch.int32, device="cuda"),
                   unique_keys=torch.full((nnz,), -7, dtype=torch.int64, device="cuda"),
                   seg_off=torch.full((nnz + 1,), -7, dtype=torch.int64, device="cuda"),
                   num_unique=torch.full((1,), -7, dtype=torch.int64, device="cuda"))
    dmt.dmt_tower_lookup_bwd_update(dw.plan, d_idx, d_off, w.batch, d_grad, lr, eps, ws, debug=dbg)
    torch.cuda.synchronize()
    return dbg


def check_bwd(w, batch_id=0):
    dw = DeviceWorkload(w, with_state=True)
    F, B = w.num_tables, w.batch
    idx, off = wl.lookup_batch(w, batch_id)
    grad = wl.grad_pooled(w, batch_id)
    # non-zero starting state so the accumulate-into-state path is exercised
    rng = np.random.default_rng(99)
    st0 = [rng.random(r).astype(np.float32) * 1e-3 for r in w.rows]
    for s, h in zip(dw.states, st0):
        s.copy_(torch.from_numpy(h))
    before = [t.clone() for t in dw.tables]
    dbg = run_bwd(dw, idx, off, grad, w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == -1

    # integer stages: bit exact
    st, sr, sp = oracle.sort_keys(F, B, idx, off)
    bag_of_pos = np.repeat(np.arange(F * B), np.diff(off))
    ut, ur, so = oracle.unique(st, sr)
    U = int(dbg["num_unique"].item())
    assert U == len(ut)
    assert np.array_equal(dbg["sorted_keys"].cpu().numpy(), (st << 32) | sr)
    assert np.array_equal(dbg["sorted_bag"].cpu().numpy(), bag_of_pos[sp].astype(np.int32))
    assert np.array_equal(dbg["unique_keys"].cpu().numpy()[:U], (ut << 32) | ur)
    assert np.array_equal(dbg["seg_off"].cpu().numpy()[:U + 1], so)

    # floating-point stages
    ref = oracle.bwd_update(dw.host_tables, w.table_dtype, st0, w.dims, w.table_to_tower, idx, off,
                            B, grad, w.lr, w.eps)
    assert np.array_equal(ref["key_table"], ut) and np.array_equal(ref["key_row"], ur)
    rtol = RTOL[w.table_dtype]
    for f in range(F):
        m = ref["key_table"] == f
        rows = ref["key_row"][m]
        D = w.dims[f]
        got_rows = to_f64(dw.tables[f][torch.from_numpy(rows).cuda()])
        want = ref["new_rows"][m][:, :D]
        if w.table_dtype != "f32":
            want = wl.decode(oracle.round_to(want, w.table_dtype), w.table_dtype)
        assert_close(got_rows, want, rtol, "%s rows of table %d" % (w.name, f))
        got_state = to_f64(dw.states[f][torch.from_numpy(rows).cuda()])
        assert_close(got_state, ref["new_state"][m].astype(np.float32), 1e-5, "state of table %d" % f)
        # rows no lookup touched are bit-identical, and so are their states
        untouched = np.ones(w.rows[f], bool)
        untouched[rows] = False
        ut_idx = torch.from_numpy(np.nonzero(untouched)[0]).cuda()
        assert torch.equal(dw.tables[f][ut_idx].view(torch.int16 if D and w.table_dtype != "f32" else torch.int32),
                           before[f][ut_idx].view(torch.int16 if w.table_dtype != "f32" else torch.int32))
        assert torch.equal(dw.states[f][ut_idx].cpu(), torch.from_numpy(st0[f])[ut_idx.cpu()])
    return dw, idx, off, grad, st0, before


def test_tiny():
    check_bwd(wl.tiny())


def test_mid_scaled_and_repeatable():
    w = wl.scaled(wl.mid(True), max_rows=20000, batch=301, num_tables=16)
    dw, idx, off, grad, st0, before = check_bwd(w)
    first_t = [t.clone() for t in dw.tables]
    first_s = [s.clone() for s in dw.states]
    # same inputs again from the same starting point: same bits
    for t, b in zip(dw.tables, before):
        t.copy_(b)
    for s, h in zip(dw.states, st0):
        s.copy_(torch.from_numpy(h))
    run_bwd(dw, idx, off, grad, w.lr, w.eps, debug=False)
    for a, b in zip(dw.tables, first_t):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for a, b in zip(dw.states, first_s):
        assert torch.equal(a, b)


@pytest.mark.parametrize("kernel", ["1", "2"])
def test_the_other_segment_reduce_kernels(kernel, monkeypatch):
    # rows of at most 128 columns take the lean walk; the wave-per-tile and lane-group walks
    # (wider rows) are reached here through the plan's switch
    monkeypatch.setenv("DMT_BWD_KERNEL", kernel)
    check_bwd(wl.scaled(wl.mid(True), max_rows=3000, batch=300, num_tables=12))
    check_bwd(wl.scaled(wl.imbalanced(), max_rows=2000, batch=400, num_tables=20))


def test_hot_rows_span_many_tiles():
    # 200 rows only: every row is hit thousands of times, runs cross many reduce tiles
    check_bwd(wl.scaled(wl.mid(True), max_rows=200, batch=512, num_tables=8))


def test_imbalanced_scaled_mixed_dims():
    check_bwd(wl.scaled(wl.imbalanced(), max_rows=5000, batch=1111, num_tables=24))


@pytest.mark.parametrize("batch", [16384, 16385, 32769, 75000])
def test_every_reduce_tile_size(batch):
    """One lookup per bag, 8 tables: 131072 (tiles of 16 records), 131080 (32), 262152 (64) and 600000
    (128) lookups, with runs that end inside a tile and runs that span many."""
    w = wl.scaled(wl.mid(True), max_rows=3000, batch=batch, num_tables=8)
    w.table_dtype = "f32"
    w.dims = [4] * 8
    w.len_dist, w.len_param, w.len_cap = "uniform", 1, 1
    check_bwd(w)


@pytest.mark.parametrize("dim", [4, 16, 32, 64, 128, 256])
@pytest.mark.parametrize("counts", [
    [5, 16 * 64], [0, 16 * 64 + 1], [7, 16 * 64 + 10],        # 63 to 65 tiles further than it starts
    [0, 16 * 65 + 1], [15, 16 * 65 + 2], [16, 16 * 66], [16 * 63, 16 * 65 + 1], [16 * 63 + 1, 16 * 66],
    [16 * 64 - 1, 16 * 129 + 2], [16 * 64, 16 * 66], [16 * 64 + 1, 16 * 64 + 15], [3, 16 * 65, 16 * 130 + 1, 4, 16 * 71],
    [16 * 200 + 9, 2, 2],
])
def test_rows_of_many_lookups_in_small_calls(dim, counts):
    """Tiles of 16 records: runs of about as many tiles as a group adds up by itself and of several times
    as many, starting at, behind and in front of a tile's and of a 64th tile's first record, one behind
    the other and up to the last record; the second table holds one run as long as its share."""
    n = sum(counts)
    w = wl.dataclasses.replace(
        wl.scaled(wl.mid(True), max_rows=10, batch=n, num_tables=2), table_dtype="f32", rows=[9, 2],
        dims=[dim] * 2, table_to_tower=[0] * 2, tm_out=[32])
    rng = np.random.default_rng(dim)
    off = np.arange(2 * n + 1, dtype=np.int64)
    idx = np.concatenate([rng.permutation(np.repeat(np.arange(len(counts)), counts)), np.ones(n)]).astype(np.int32)
    dw = DeviceWorkload(w, with_state=True, max_nnz=2 * n)
    grad = wl.grad_pooled(w)
    run_bwd(dw, idx, off, grad, w.lr, w.eps, debug=False)
    assert dw.dmt.dmt_last_device_error(dw.plan) == -1
    ref = oracle.bwd_update(dw.host_tables, "f32", [np.zeros(r, np.float32) for r in w.rows], w.dims, w.table_to_tower,
                            idx, off, n, grad, w.lr, w.eps)
    for f in range(2):
        m = ref["key_table"] == f
        rows = torch.from_numpy(ref["key_row"][m]).cuda()
        assert_close(to_f64(dw.tables[f][rows]), ref["new_rows"][m][:, :dim], 1e-5, "rows")
        # (a sum of n terms of either sign: its float32 error is a few units of the terms' root sum of squares)
        assert_close(to_f64(dw.states[f][rows]), ref["new_state"][m], 2e-5, "state")


@pytest.mark.parametrize("rows,lens", [
    ([1, 1], [900, 2]), ([1022, 3], [1000, 1]), ([1024, 5, 1023], [2049, 0, 1]),      # one launch: 1, 10 and 11 bits
    ([1, 1], [9000, 2]),                            # one bit of row id
    ([1022, 3], [9000, 1]),                         # 10 bits: one pass
    ([1024, 5, 1023], [8193, 0, 1]),                # 11 bits: two passes; blocks of one record
    ([50] * 400, [20] * 400),                       # bags of many tables in one block of bwd_bag_samples; narrow digits
    ([1 << 20, 40], [40000, 3]),                    # 21 bits: three passes; 20 blocks in one table
    ([3000, 70000, 9], [(1 << 18), 1, (1 << 18) - 1]),   # as many lookups as wide digits take
    ([3000, 70000, 9], [(1 << 18), 1, 1 << 18]),    # one more: narrow digits
])
def test_sort_digit_widths(rows, lens):
    """Two bags a table, the first with two thirds of the table's lookups: the sorted order is the
    stable order of (table, row), whatever the digits' width and the tables' share."""
    F = len(rows)
    w = wl.dataclasses.replace(
        wl.scaled(wl.mid(True), max_rows=10, batch=2, num_tables=F), table_dtype="f32", rows=rows,
        dims=[16] * F, table_to_tower=[0] * F, tm_out=[32])
    per_bag = np.array([c for n in lens for c in (n - n // 3, n // 3)], dtype=np.int64)
    off = np.concatenate([[0], np.cumsum(per_bag)])
    rng = np.random.default_rng(7)
    idx = np.concatenate([(r * rng.random(n) ** 3).astype(np.int32) for r, n in zip(rows, lens)])
    dw = DeviceWorkload(w, with_state=True, max_nnz=sum(lens))
    dbg = run_bwd(dw, idx, off, wl.grad_pooled(w), w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == -1
    key = (np.repeat(np.arange(F, dtype=np.int64), lens) << 32) | idx
    order = np.argsort(key, kind="stable")
    bag = np.repeat(np.arange(2 * F), per_bag)
    assert np.array_equal(dbg["sorted_keys"].cpu().numpy(), key[order])
    assert np.array_equal(dbg["sorted_bag"].cpu().numpy(), bag[order])


@pytest.mark.parametrize("rows", [[200, 1], [1 << 12, 9], [1 << 20, 70000, 3]])      # 1, 2 and 3 passes of narrow digits
@pytest.mark.parametrize("batch,mean,longest", [
    (3, 0.0, 5000), (700, 0.4, 5000),                # one launch sorts these,
    (3, 0.0, 9000), (700, 0.4, 9000),                # wide digits these,
    (3, 0.0, 600_000), (700, 0.4, 600_000),          # and narrow ones these and the others
    (1025, 900.0, 0), (65536, 5.0, 0), (65537, 5.0, 0),
])
def test_samples_of_the_sorted_lookups(rows, batch, mean, longest):
    """Samples of 16 bits (up to 65536) and of 32, bags of a table with fewer, as many and more samples than a block of
    bwd_bag_samples takes, most bags empty or one holding most lookups: order and samples are exact."""
    F = len(rows)
    w = wl.dataclasses.replace(
        wl.scaled(wl.mid(True), max_rows=10, batch=batch, num_tables=F), table_dtype="f32", rows=rows,
        dims=[4] * F, table_to_tower=[0] * F, tm_out=[32])
    rng = np.random.default_rng(batch)
    per_bag = rng.poisson(mean, F * batch).astype(np.int64)
    if longest:
        per_bag[[0, F * batch - 1, F * batch // 2]] = [longest, 1, 3]
    off = np.concatenate([[0], np.cumsum(per_bag)])
    lens = per_bag.reshape(F, batch).sum(1)
    idx = np.concatenate([(r * rng.random(n) ** 3).astype(np.int32) for r, n in zip(rows, lens)])
    dw = DeviceWorkload(w, with_state=True, max_nnz=len(idx))
    dbg = run_bwd(dw, idx, off, wl.grad_pooled(w), w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == -1
    key = (np.repeat(np.arange(F, dtype=np.int64), lens) << 32) | idx
    order = np.argsort(key, kind="stable")
    assert np.array_equal(dbg["sorted_keys"].cpu().numpy(), key[order])
    assert np.array_equal(dbg["sorted_bag"].cpu().numpy(), np.repeat(np.arange(F * batch), per_bag)[order])


@pytest.mark.parametrize("rows", [[200, 1], [1 << 12, 9], [1 << 20, 70000, 3]])      # 1, 2 and 3 passes
@pytest.mark.parametrize("share", [1e-6, 0.3])
def test_ids_outside_their_table_in_narrow_digits(rows, share):
    """More than 2^19 lookups: they sort behind the table's rows in the order of the lookups, touch no row, and the first
    is reported."""
    F, batch, n = len(rows), 500, 300_000
    w = wl.dataclasses.replace(
        wl.scaled(wl.mid(True), max_rows=10, batch=batch, num_tables=F), table_dtype="f32", rows=rows,
        dims=[4] * F, table_to_tower=[0] * F, tm_out=[32])
    rng = np.random.default_rng(F)
    off = np.arange(F * batch + 1, dtype=np.int64) * (n // batch)
    table = np.repeat(np.arange(F, dtype=np.int64), n)
    size = np.array(rows)[table]
    idx = (size * rng.random(F * n) ** 3).astype(np.int32)
    outside = rng.random(F * n) < share
    outside[[7, F * n - 1]] = True
    idx[outside] = np.where(rng.random(outside.sum()) < 0.5, size[outside], -1 - size[outside]).astype(np.int32)
    dw = DeviceWorkload(w, with_state=True, max_nnz=F * n)
    before = [t.clone() for t in dw.tables]
    dbg = run_bwd(dw, idx, off, wl.grad_pooled(w), w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == np.flatnonzero(outside)[0]
    order = np.argsort(table << 32 | np.where(outside, size, idx), kind="stable")
    assert np.array_equal(dbg["sorted_keys"].cpu().numpy(), np.where(outside, -1, table << 32 | idx)[order])
    assert np.array_equal(dbg["sorted_bag"].cpu().numpy(), (np.arange(F * n) // (n // batch))[order])
    for f in range(F):
        hit = np.zeros(rows[f], bool)
        hit[idx[(table == f) & ~outside]] = True
        same = (dw.tables[f] == before[f]).all(dim=1).cpu().numpy()
        assert not same[hit].any() and same[~hit].all()


@pytest.mark.parametrize("rows,lens,batch", [
    ([1000, 7, 1], [1, 0, 64], 3), ([1023, 1024, 40], [1024, 1025, 7168 - 2049], 200), ([1 << 20], [7168], 2048),
    ([1 << 20], [7168], 2049), ([1 << 20], [7169], 100),     # either line's other side: several launches
    ([30000] * 70, [13] * 70, 1), ([1 << 21, 3], [63, 65], 2048),
])
@pytest.mark.parametrize("bags", ["even", "first", "last", "sparse"])
def test_sort_of_few_lookups(rows, lens, batch, bags):
    """One launch sorts them: one to three passes, tables of no, one and many lookups around a wave's and a step's,
    samples even, all in the first or last bag, or with most bags empty; ids outside their table behind the others."""
    F = len(rows)
    w = wl.dataclasses.replace(
        wl.scaled(wl.mid(True), max_rows=10, batch=batch, num_tables=F), table_dtype="f32", rows=rows,
        dims=[4] * F, table_to_tower=[0] * F, tm_out=[32])
    rng = np.random.default_rng(len(rows) + batch)
    per_bag = np.zeros((F, batch), np.int64)
    for f, n in enumerate(lens):
        at = {"even": np.arange(n) % batch, "first": np.zeros(n, int), "last": np.full(n, batch - 1),
              "sparse": rng.integers(0, max(1, batch // 50), n) * 50 % batch}[bags]
        np.add.at(per_bag[f], at, 1)
    per_bag = per_bag.reshape(-1)
    off = np.concatenate([[0], np.cumsum(per_bag)])
    idx = np.concatenate([(r * rng.random(n) ** 3).astype(np.int32) for r, n in zip(rows, lens)])
    outside = rng.random(len(idx)) < 0.01
    idx[outside] = -5
    dw = DeviceWorkload(w, with_state=True, max_nnz=len(idx))
    dbg = run_bwd(dw, idx, off, wl.grad_pooled(w), w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == (np.flatnonzero(outside)[0] if outside.any() else -1)
    table = np.repeat(np.arange(F, dtype=np.int64), lens)
    order = np.argsort(table << 32 | np.where(outside, np.array(rows)[table], idx), kind="stable")
    assert np.array_equal(dbg["sorted_keys"].cpu().numpy(), np.where(outside, -1, table << 32 | idx)[order])
    assert np.array_equal(dbg["sorted_bag"].cpu().numpy(), np.repeat(np.arange(F * batch), per_bag)[order])


@pytest.mark.parametrize("dims", [[32, 64], [64], [32], [256]])
def test_narrow_and_wide_rows(dims):
    """Dims up to 128 run the lean walk, 256 the wave-per-tile kernel."""
    w = wl.scaled(wl.imbalanced(), max_rows=3000, batch=400, num_tables=12)
    w.dims = [dims[f % len(dims)] for f in range(12)]
    check_bwd(w)


@pytest.mark.parametrize("widest", [136, 160, 200, 248])
def test_widest_row_between_128_and_256_columns(widest):
    """Mixed widths whose widest row is neither 128 nor 256 columns take the lane-group walk with
    64-lane groups of which only widest / 4 lanes hold columns; the records of the other lanes
    count like any other (they once did not: their gradients were dropped)."""
    w = wl.scaled(wl.imbalanced(), max_rows=700, batch=150, num_tables=9)
    w.dims = [widest, 64, 16, 128, widest, 32, 8, 96, 24]
    check_bwd(w)


def test_large_scaled_bf16():
    w = wl.scaled(wl.large(), max_rows=30000, batch=130, num_tables=40)
    w.backward = True
    check_bwd(w)


def test_many_small_tables_some_without_lookups():
    """300 tables (more than one pass of the sort-block map's 256-table chunks), a few rows each,
    Poisson(0.3) bag lengths so that many tables have no lookup at all in a batch of 3."""
    base = wl.scaled(wl.imbalanced(), max_rows=60, batch=3, num_tables=100)
    w = wl.dataclasses.replace(
        base, rows=[7 + (f * 13) % 50 for f in range(300)], dims=[32] * 300,
        table_to_tower=[f // 25 for f in range(300)], tm_out=[128] * 12, len_dist="poisson",
        len_param=0.3, len_cap=3, zipf_alpha=None)
    check_bwd(w)


def test_empty_batch_is_a_no_op():
    w = wl.scaled(wl.mid(True), max_rows=100, batch=9, num_tables=8)
    dw = DeviceWorkload(w, with_state=True)
    before = [t.clone() for t in dw.tables]
    off = np.zeros(w.num_tables * w.batch + 1, dtype=np.int64)
    dbg = run_bwd(dw, np.zeros(0, np.int32), off, wl.grad_pooled(w), 0.01, 1e-8)
    assert int(dbg["num_unique"].item()) == 0 and int(dbg["seg_off"][0].item()) == 0
    for a, b in zip(dw.tables, before):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_out_of_range_ids_are_skipped():
    w = wl.scaled(wl.mid(True), max_rows=100, batch=16, num_tables=8)
    dw = DeviceWorkload(w, with_state=True)
    idx, off = wl.lookup_batch(w)
    grad = wl.grad_pooled(w)
    bad = idx.copy()
    bad[[5, 700]] = [100, -1]
    dbg = run_bwd(dw, bad, off, grad, w.lr, w.eps)
    assert dw.dmt.dmt_last_device_error(dw.plan) == 5
    keep = np.ones(len(idx), bool); keep[[5, 700]] = False
    lens = np.diff(off)
    bag_of = np.repeat(np.arange(len(lens)), lens)
    new_off = np.concatenate([[0], np.cumsum(np.bincount(bag_of[keep], minlength=len(lens)))])
    st0 = [np.zeros(r, np.float32) for r in w.rows]
    ref = oracle.bwd_update(dw.host_tables, w.table_dtype, st0, w.dims, w.table_to_tower,
                            idx[keep], new_off, w.batch, grad, w.lr, w.eps)
    assert int(dbg["num_unique"].item()) == len(ref["key_row"])
    for f in range(w.num_tables):
        m = ref["key_table"] == f
        rows = ref["key_row"][m]
        want = wl.decode(oracle.round_to(ref["new_rows"][m][:, :w.dims[f]], "f16"), "f16")
        assert_close(to_f64(dw.tables[f][torch.from_numpy(rows).cuda()]), want, 2e-2, "rows")


@pytest.mark.parametrize("case", ["first_not_zero", "descending", "last_not_nnz", "beyond_nnz"])
def test_malformed_offsets_update_nothing_and_are_reported(case):
    # the host cannot see device offsets; bwd_bag_samples checks them and the update is skipped
    w = wl.scaled(wl.mid(True), max_rows=100, batch=16, num_tables=8)
    dw = DeviceWorkload(w, with_state=True)
    idx, off = wl.lookup_batch(w)
    grad = wl.grad_pooled(w)
    bad = off.copy()
    nbags = len(off) - 1
    if case == "first_not_zero":
        bad[0], where = 3, 0
    elif case == "descending":
        bad[41], where = bad[40] - 1 if bad[40] > 0 else bad[42] + 1, 40
        if bad[41] > bad[42]:
            where = 41
    elif case == "last_not_nnz":
        bad[-1], where = len(idx) - 2, nbags - 1
    else:
        bad[-1], where = len(idx) + 5, nbags - 1
    before = [t.clone() for t in dw.tables]
    run_bwd(dw, idx, bad, grad, w.lr, w.eps, debug=False)
    with pytest.raises(dw.dmt.DmtError) as e:
        dw.dmt.dmt_last_device_error(dw.plan)
    assert e.value.code == 1 and e.value.position == where           # DMT_EINVAL, first bad bag
    for a, b, s in zip(dw.tables, before, dw.states):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert int((s != 0).sum()) == 0
    # the record is cleared and a well-formed call works afterwards
    run_bwd(dw, idx, off, grad, w.lr, w.eps, debug=False)
    assert dw.dmt.dmt_last_device_error(dw.plan) == -1
    assert sum(int((s != 0).sum()) for s in dw.states) > 0


@pytest.mark.parametrize("case", ["first_not_zero", "descending", "last_not_nnz", "beyond_nnz"])
def test_malformed_offsets_of_a_call_that_several_launches_sort(case, monkeypatch):
    """The same with 19 K lookups: past the line of bwd_sort_small, which makes the checks of the smaller call."""
    scaled = wl.scaled
    monkeypatch.setattr(wl, "scaled", lambda w, **sizes: scaled(w, **dict(sizes, batch=120)))
    test_malformed_offsets_update_nothing_and_are_reported(case)


def test_malformed_offsets_of_many_tables_stay_inside_the_workspace():
    """Tables whose first bags start at 0, nnz, 0, nnz ...: added up, the tables' lengths pass 2^32, and blocks that
    start from such a sum would list 16384 sort blocks where the launch has 9216.  Nothing is touched, inside the
    tables or behind the workspace."""
    import paper_2403_00877_amd as dmt
    F, nnz, dim, rows = 1024, 1 << 24, 4, 16
    off = torch.zeros(F + 1, dtype=torch.int64)
    off[1::2] = nnz
    tabs = torch.ones(F, rows, dim, device="cuda")
    states = torch.zeros(F, rows, device="cuda")
    plan = dmt.dmt_plan_create([rows] * F, [dim] * F, "f32", 1, [0] * F, 1, nnz)
    dmt.dmt_plan_bind(plan, list(tabs), list(states))
    need = dmt.dmt_bwd_workspace_bytes(plan, 1, nnz)
    ws = torch.full((need + 4096,), 171, dtype=torch.uint8, device="cuda")
    idx = torch.zeros(nnz, dtype=torch.int32, device="cuda")
    grad = torch.ones(F * dim, device="cuda")
    dmt.dmt_tower_lookup_bwd_update(plan, idx, off.cuda(), 1, grad, 0.01, 1e-8, ws[:need])
    with pytest.raises(dmt.DmtError) as e:
        dmt.dmt_last_device_error(plan)
    assert e.value.code == 1 and e.value.position == 1               # DMT_EINVAL, first bad bag
    assert bool((ws[need:] == 171).all()) and bool((tabs == 1).all()) and bool((states == 0).all())


def _degenerate(ids_of):
    w = wl.scaled(wl.mid(True), max_rows=5000, batch=64, num_tables=2)
    w.table_to_tower = [0, 0]
    w.tm_out = [256]
    dw = DeviceWorkload(w, with_state=True)
    lens = np.full(2 * 64, 30, dtype=np.int64)
    off = np.concatenate([[0], np.cumsum(lens)])
    idx = ids_of(int(off[-1])).astype(np.int32)
    grad = wl.grad_pooled(w)
    dbg = run_bwd(dw, idx, off, grad, w.lr, w.eps)
    st0 = [np.zeros(r, np.float32) for r in w.rows]
    ref = oracle.bwd_update(dw.host_tables, w.table_dtype, st0, w.dims, w.table_to_tower, idx, off,
                            w.batch, grad, w.lr, w.eps)
    assert int(dbg["num_unique"].item()) == len(ref["key_row"])
    for f in range(2):
        m = ref["key_table"] == f
        rows = torch.from_numpy(ref["key_row"][m]).cuda()
        want = wl.decode(oracle.round_to(ref["new_rows"][m][:, :128], "f16"), "f16")
        assert_close(to_f64(dw.tables[f][rows]), want, 2e-2, "rows")
        assert_close(to_f64(dw.states[f][rows]), ref["new_state"][m], 1e-5, "state")


def test_every_lookup_hits_the_same_row():
    # one run per table as long as the table's whole record range: 15 reduce tiles chained
    _degenerate(lambda n: np.full(n, 17))


def test_every_lookup_hits_a_different_row():
    # no duplicates at all: every run has length one
    _degenerate(lambda n: np.arange(n) % 1920 + (np.arange(n) // 1920) * 0)


@pytest.mark.parametrize("tables,batch,length", [(1, 64, 9), (1, 520, 63), (3, 129, 16), (3, 511, 33), (8, 257, 8),
                                                 (2, 1030, 64), (26, 300, 13)])
def test_sort_blocks_of_every_size(tables, batch, length):
    """Sort blocks of 512 records (two a thread; five in the last but one case), tables that end inside, at and
    past a block's edge: the sorted order against a stable sort of the ids."""
    _sorted_order([batch * length] * tables, batch, [length] * tables)


# records a thread by table (of at least the call's least): a table of L lookups gets ceil(L / 16384), 2 to 8
@pytest.mark.parametrize("lens", [
    [40_000], [60_000], [90_000], [100_000], [110_000], [130_000],           # 3, 4, 6, 7, 7 and 8
    [16_384 * 2], [16_384 * 2 + 1], [16_384 * 5], [16_384 * 5 + 1],          # the lines between two sizes
    [500, 126_000, 0, 511, 513, 1, 2000, 4096],                              # nearly all of a call in one table
    [1, 1, 300_000, 33_000, 70_000, 7],                                      # several sizes in one call
    [5] * 40 + [130_001] + [1500] * 23,
    [262_144, 262_144], [524_288], [524_289],                                # least of 8; the last wide digits, narrow ones
])
def test_sort_blocks_follow_each_table(lens):
    _sorted_order(lens, 64)


@pytest.mark.parametrize("tables,each", [(60, 90), (64, 400), (200, 40), (300, 433)])
def test_sort_blocks_where_counts_are_short_of_room(tables, each):
    """Many tables of narrow rows: fewer and larger sort blocks, or narrow digits."""
    _sorted_order([each] * tables, 32)


def _sorted_order(lens, batch, bag=None):
    """Table t has lens[t] lookups, spread over its bags as evenly as they go (or bag[t] each)."""
    import paper_2403_00877_amd as dmt
    tables, nnz, dim = len(lens), sum(lens), 8
    rows = [5000 + 37 * f for f in range(tables)]
    g = torch.Generator(device="cuda")
    g.manual_seed(tables)
    idx = torch.cat([torch.randint(0, r, (n,), generator=g, device="cuda") for r, n in zip(rows, lens)]).to(torch.int32)
    per = torch.tensor(lens, device="cuda").repeat_interleave(batch)
    b = torch.arange(batch, device="cuda").repeat(tables)
    counts = per // batch + (b < per % batch)
    off = torch.zeros(tables * batch + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(counts, 0)
    assert bag is None or torch.equal(counts, torch.tensor(bag, device="cuda").repeat_interleave(batch))
    tabs = [torch.zeros(r, dim, device="cuda") for r in rows]
    states = [torch.zeros(r, device="cuda") for r in rows]
    plan = dmt.dmt_plan_create(rows, [dim] * tables, "f32", 1, [0] * tables, batch, nnz)
    dmt.dmt_plan_bind(plan, tabs, states)
    grad = torch.randn(batch * tables * dim, generator=g, device="cuda")
    ws = torch.empty(dmt.dmt_bwd_workspace_bytes(plan, batch, nnz), dtype=torch.uint8, device="cuda")
    keys = torch.empty(nnz, dtype=torch.int64, device="cuda")
    bags = torch.empty(nnz, dtype=torch.int32, device="cuda")
    dmt.dmt_tower_lookup_bwd_update(plan, idx, off, batch, grad, 0.01, 1e-8, ws,
                                    debug=dict(sorted_keys=keys, sorted_bag=bags))
    table = torch.arange(tables, device="cuda").repeat_interleave(torch.tensor(lens, device="cuda"))
    ref, order = torch.sort((table << 32) | idx.to(torch.int64), stable=True)
    assert torch.equal(keys, ref)
    which = torch.arange(tables * batch, device="cuda").repeat_interleave(counts)
    assert torch.equal(bags.to(torch.int64), which[order])
