"""Edges of the whole-wave row kernels against the oracle: product counts at
the register and sort limits, column spans at the bitmap's, buckets at their
fullest, empty B rows, more A entries than lanes.  Structure identical,
values within the repository's bounds (1e-12 FP64, 1e-5 FP32 times the sum of
|a||b|: a row of at most 1024 FP64 additions is off by less than 1024 2^-53)."""
import ctypes

import numpy as np
import pytest

from paper_2112_10037_amd import binding, gen, learned

from gpu_util import TOL, check_full, check_rows, run, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    hh = binding.Handle(0)
    yield hh
    hh.close()


def _csr(rows, ncols, rng, dtype):
    rp = np.zeros(len(rows) + 1, np.int64)
    rp[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate([np.sort(np.asarray(r)) for r in rows]).astype(np.int32) if rp[-1] else np.zeros(0, np.int32)
    return gen.CSR(len(rows), ncols, rp, col, (2 * rng.random(int(rp[-1])) - 1).astype(dtype))


def _lengths(total, na):
    """na B-row lengths that add up to total, some of them 0 when na allows."""
    out = np.full(na, total // na)
    out[: total % na] += 1
    return out


# name: (total products, A entries, distinct columns to draw from, first and last column)
CASES = {
    "narrow_full": (768, 64, 500, 0, 39_999),
    "narrow_over": (769, 64, 500, 0, 39_999),
    "narrow_one_entry": (65, 1, 65, 7, 8_000),
    "narrow_step": (256, 32, 240, 3, 300),
    "narrow_step_over": (257, 32, 240, 3, 300),
    "span_last_narrow": (200, 20, 180, 5, 5 + 43_007),
    "span_first_wide": (200, 20, 180, 5, 5 + 43_008),
    "wide_sort_full": (512, 40, 250, 0, 999_999),
    "wide_sort_over": (513, 40, 250, 0, 999_999),
    "wide_sort_full_512": (768, 48, 500, 0, 999_999),
    "wide_sort_over_512": (769, 48, 500, 0, 999_999),
    "wide_one_step": (64, 8, 64, 0, 2_000_000),
    "wide_lanes_plus_one": (65, 13, 65, 0, 2_000_000),
    "symbolic_256": (256, 30, 4000, 0, 900_000),
    "symbolic_257": (257, 30, 4000, 0, 900_000),
    "symbolic_512": (512, 30, 40_000, 0, 900_000),
    "symbolic_513": (513, 30, 40_000, 0, 900_000),
    "symbolic_1024": (1024, 50, 900, 0, 900_000),
    "entries_64": (200, 64, 150, 0, 900_000),
    "entries_65": (200, 65, 150, 0, 900_000),
    "entries_65_narrow": (200, 65, 150, 0, 900),
}


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("name", sorted(CASES))
def test_row_kernel_edges(h, name, dtype):
    total, na, pool, lo, hi = CASES[name]
    rng = np.random.default_rng(total * 131 + na)
    n = hi + 1
    arows, brows = [], []
    for _ in range(24):
        cols = np.unique(np.concatenate([[lo, hi], rng.integers(lo, hi + 1, size=4 * pool)]))
        cols = np.sort(np.concatenate([[lo, hi], rng.permutation(cols[1:-1])[: pool - 2]]))
        first = len(brows)
        # empty B rows first, in the middle and last, where the entries leave room
        empty = [0, na // 2, na - 1] if 8 <= na < 64 else []
        lens = np.zeros(na, np.int64)
        lens[[i for i in range(na) if i not in empty]] = _lengths(total, na - len(empty))
        ends = int(np.argmax(lens >= 2))             # the B row that holds the span's ends
        for i, length in enumerate(lens):
            if i == ends:
                pick = np.concatenate([[0, len(cols) - 1], 1 + rng.permutation(len(cols) - 2)[: length - 2]])
            else:
                pick = rng.permutation(len(cols))[:length]
            brows.append(cols[pick])
        arows.append(np.arange(first, first + na))
    A = _csr(arows, len(brows), rng, dtype)
    B = _csr(brows, n, rng, dtype)
    check_full(h, A, B)
    check_full(h, A, B, tuning=(1, 0, 4096, 128, 8))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("same", [24, 25])
def test_row_kernel_fullest_bucket(h, same, dtype):
    """`same` products share one column, the others spread over two million."""
    rng = np.random.default_rng(same)
    arows, brows = [], []
    for _ in range(12):
        first = len(brows)
        other = 10 + rng.permutation(2_000_000)[: 9 * same]
        for i in range(same):
            brows.append(np.concatenate([[3], other[9 * i: 9 * i + 9]]))
        arows.append(np.arange(first, first + same))
    A = _csr(arows, len(brows), rng, dtype)
    B = _csr(brows, 2_000_010, rng, dtype)
    check_full(h, A, B)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_row_kernel_many_rows_per_wave(h, dtype):
    """More rows than waves, long, short and empty ones in turn, so that every
    wave loads rows of one path while it works on another's."""
    rng = np.random.default_rng(5)
    k = rng.choice([0, 1, 9, 16, 30, 70], size=24_000, p=[0.1, 0.1, 0.2, 0.3, 0.2, 0.1])
    A = gen.erdos_renyi(24_000, 5_000, k, seed=6, dtype=dtype)
    kb = rng.integers(0, 14, size=5_000)
    check_full(h, A, gen.erdos_renyi(5_000, 300_000, kb, seed=7, dtype=dtype))
    check_full(h, A, gen.erdos_renyi(5_000, 3_000, kb, seed=8, dtype=dtype))


# name: (total products, A entries, distinct columns, first and last column)
SORT_CASES = {
    "cap_128": (1024, 40, 900, 0, 1_500_000),
    "over_128": (1025, 40, 900, 0, 1_500_000),
    "cap_256": (2048, 200, 1900, 0, 3000),
    "over_256": (2049, 200, 1900, 0, 3000),
    "cap_512": (4096, 300, 3900, 0, 1_500_000),
    "over_512": (4097, 300, 3900, 0, 1_500_000),
    "entries_128": (900, 128, 850, 0, 50_000),
    "entries_129": (900, 129, 850, 0, 50_000),
    "entries_767": (900, 767, 850, 0, 50_000),
    "entries_768": (900, 768, 850, 0, 50_000),
    "entries_3071": (3900, 3071, 2900, 0, 1_500_000),
    "entries_3072": (3900, 3072, 2900, 0, 1_500_000),
    "one_entry": (3000, 1, 3000, 0, 1_500_000),
    "apart": (1500, 10, 60_000, 0, 1_500_000),
    "bucket_256": (3000, 256, 2500, -1, 1_500_000),
    "bucket_257": (3000, 257, 2500, -1, 1_500_000),
}


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("name", sorted(SORT_CASES))
def test_sort_kernel_edges(h, name, dtype):
    """Rows of 513 to 4096 outputs at the workgroup sort's limits of products,
    A entries and products in one bucket (first column -1: every B row starts
    with column 0), with empty B rows among the entries."""
    total, na, pool, lo, hi = SORT_CASES[name]
    rng = np.random.default_rng(total + 7 * na)
    arows, brows = [], []
    for _ in range(9):
        first = len(brows)
        # an empty B row before, between and after; they are entries too
        lens = np.zeros(na, np.int64)
        full = [i for i in range(na) if not (16 < na < 900 and lo >= 0 and i in (0, na // 3, na - 1))]
        lens[full] = _lengths(total, len(full))
        cols = 1 + np.sort(rng.permutation(hi - 1)[:pool])
        for length in lens:
            pick = cols[rng.permutation(pool)[: length - (lo < 0)]] if length else cols[:0]
            brows.append(np.concatenate([[0], pick]) if lo < 0 else pick)
        arows.append(np.arange(first, first + na))
    A = _csr(arows, len(brows), rng, dtype)
    B = _csr(brows, hi + 1, rng, dtype)
    check_full(h, A, B)


# name: (total products, A entries, distinct columns, columns of B)
LIST_CASES = {
    "cap_2048": (2048, 100, 1800, 1_200_000),
    "over_2048": (2049, 100, 1800, 1_200_000),
    "cap_8192": (8192, 700, 7000, 1_200_000),
    "over_8192": (8193, 700, 7000, 1_200_000),
    "cap_16384": (16384, 1500, 12_000, 1_200_000),
    "over_16384": (16385, 1500, 12_000, 1_200_000),
    "single_entries": (5000, 5000, 4000, 1_200_000),
    "one_entry": (5000, 1, 5000, 1_200_000),
    "width_bounds": (9000, 40, 3000, 3000),
    "width_bounds_16k": (40_000, 40, 12_000, 12_000),
}


@pytest.mark.parametrize("name", sorted(LIST_CASES))
def test_list_kernel_edges(h, name):
    """Symbolic rows of 1025 to 16,384 products at the workgroup lists' limits,
    rows bounded by B's width rather than their products, and both numeric
    thresholds that leave window records."""
    total, na, pool, n = LIST_CASES[name]
    rng = np.random.default_rng(total + na)
    arows, brows = [], []
    for _ in range(7):
        first = len(brows)
        cols = np.sort(rng.permutation(n)[:pool])
        for length in _lengths(total, na):
            brows.append(cols[rng.permutation(pool)[:length]])
        arows.append(np.arange(first, first + na))
    A = _csr(arows, len(brows), rng, np.float32)
    B = _csr(brows, n, rng, np.float32)
    check_full(h, A, B)
    check_full(h, A, B, tuning=(1, 0, 512, 128, 8))
    nnz = h.symbolic(binding.DeviceCSR.from_host(A), binding.DeviceCSR.from_host(B))
    import oracle
    assert np.array_equal(nnz[0].cpu().numpy(), oracle.row_nnz(A, B))


@pytest.mark.parametrize("wide", [1, 300])
def test_fused_sums_of_long_rows(h, wide):
    """The statistics pass's three sums: rows around 4 and 8 A entries (heads),
    around 32 and 512 (eight lanes), and from 513 on (the workgroup), in tiles
    of 256 rows with one or with every row long; last tile partly filled."""
    rng = np.random.default_rng(wide)
    k = rng.choice([0, 3, 4, 5, 8, 9, 31, 32, 33, 64, 65], size=900)
    k[rng.permutation(900)[:6]] = [511, 512, 513, 1024, 1025, 4000]
    k[256: 256 + wide] = 513 + rng.integers(0, 1100, size=wide)
    A = gen.erdos_renyi(900, 6_000, k, seed=9)
    B = gen.erdos_renyi(6_000, 40_000, rng.choice([0, 0, 0, 1, 1, 2, 7], size=6_000), seed=10)
    check_full(h, A, B)


@pytest.mark.parametrize("ncols", [33, 64, 65, 128, 511, 1000, 1024, 43_008, 43_009, 900_000])
def test_symbolic_rows_past_the_registers(h, ncols):
    """More products than a row's columns allow in registers, or more A entries
    than lanes: windows of 1024 products entered, filled and passed, B rows
    that are empty, short or as long as B is wide, the bitmap's last column and
    the first width without it."""
    rng = np.random.default_rng(ncols)
    kb = rng.choice([0, 1, 2, 9, 30, min(ncols, 900)], size=600, p=[0.2, 0.3, 0.2, 0.2, 0.08, 0.02])
    B = gen.erdos_renyi(600, ncols, np.minimum(kb, ncols), seed=41)
    B.col[B.row_ptr[1:][np.diff(B.row_ptr) > 0] - 1] = ncols - 1
    ka = rng.choice([1, 7, 20, 63, 64, 65, 90, 128, 129, 300], size=700)
    A = gen.erdos_renyi(700, 600, ka, seed=42)
    check_full(h, A, B)
    check_full(h, A, B, tuning=(1, 0, 4096, 1024, 8))


@pytest.mark.parametrize("rows", [16_383, 16_384, 17_001])
@pytest.mark.parametrize("ncols", [64, 65, 128, 129, 60_000])
def test_many_short_rows(h, ncols, rows):
    """Both sides of the row count from which the shortest whole-wave bin takes
    several rows a wave, and of the column counts below which the symbolic pass
    does; every row has 33 to 64 outputs, or more where B is wide enough."""
    rng = np.random.default_rng(rows)
    A = gen.erdos_renyi(rows, 700, rng.choice([6, 7], size=rows), seed=51)
    B = gen.erdos_renyi(700, ncols, 8, seed=52)
    check_full(h, A, B)
    A = gen.erdos_renyi(rows, 700, rng.choice([8, 30], size=rows), seed=53)
    check_full(h, A, B)


@pytest.mark.parametrize("first", ["empty", "entries"])
@pytest.mark.parametrize("total,na", [(900, 40), (3900, 300), (7000, 60), (12_000, 60)])
def test_workgroup_rows_start_without_a_walk(h, total, na, first):
    """Every row in one bin of the workgroup kernels, so they are taken in
    their natural order, and a workgroup's first row takes no turn of the walk
    over A entries: empty rows, or rows of more A entries (most select empty B
    rows) than the numeric sort takes.  More rows than a first round has."""
    rng = np.random.default_rng(total)
    ncols, rows = 2_000_000, 2600
    none = np.arange(4000, 8000)                     # empty B rows
    lens = _lengths(total, na)
    brows = [np.sort(rng.integers(0, ncols, size=2 * length))[::2] for length in np.tile(lens, 4000 // na)]
    brows = [np.unique(r) for r in brows] + [np.zeros(0, np.int64)] * (8000 - na * (4000 // na))
    arows = []
    for i in range(rows):
        base = int(rng.integers(0, 4000 // na)) * na
        row = np.arange(base, base + na)
        if i < 1100 or i % 7 == 0:                   # (at most four workgroups a compute unit start on the first ones)
            row = row[:0] if first == "empty" else np.concatenate([row, none])
        arows.append(row)
    A = _csr(arows, len(brows), rng, np.float32)
    B = _csr(brows, ncols, rng, np.float32)
    C = run(h, A, B)
    check_rows(C, A, B, [0, 1, 7, 1099, 1100, 1101, 2598, 2599])
    import oracle
    nnz = h.symbolic(binding.DeviceCSR.from_host(A), binding.DeviceCSR.from_host(B))[0]
    assert np.array_equal(nnz.cpu().numpy(), oracle.row_nnz(A, B))
    assert np.array_equal(np.diff(C.row_ptr.cpu().numpy()), oracle.row_nnz(A, B))


@pytest.fixture(scope="module")
def wide():
    """A handle that keeps positions in B as if B had 2^32 entries or more."""
    hh = binding.Handle(0)
    f = hh._lib.msp_internal_set_narrow_positions
    f.argtypes = [ctypes.c_void_p, ctypes.c_longlong]
    f(hh._h, 0)
    yield hh
    hh.close()


@pytest.mark.parametrize("name", sorted(LIST_CASES))
def test_list_kernel_edges_with_wide_positions(wide, name):
    test_list_kernel_edges(wide, name)


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("ncols", [1_200_000, 20_000])
def test_lists_side_by_side_with_wide_positions(wide, ncols, batch):
    """Few rows in each of the symbolic lists' bins and in the bitmap bin, which
    run at the same time, with more columns than the LDS bitmap holds."""
    rng = np.random.default_rng(ncols)
    B = gen.erdos_renyi(40_000, ncols, 25, seed=61)
    A = gen.erdos_renyi(300, 40_000, rng.choice([3, 50, 200, 400, 900], size=300), seed=62)
    if not batch:
        check_full(wide, A, B)
        return
    plan = binding.Batch(wide, *[binding.PackedBatch.from_host([x, x]) for x in (A, B)])
    plan.execute()
    import oracle
    ref = oracle.spgemm(A, B)
    for p in range(2):
        got = plan.result(p).to_host()
        oracle.compare(got.row_ptr, got.col, got.val, ref, 1e-12)
    plan.close()


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("total,na,lo,hi", [(200, 20, 0, 40_000), (300, 20, 0, 2_000_000), (600, 40, 0, 2_000_000),
                                            (900, 40, 0, 2_000_000), (1900, 100, 0, 3000), (3900, 300, 0, 2_000_000)])
def test_counts_that_are_too_high_are_reported(h, total, na, lo, hi, dtype):
    """Row counts of a symbolic pass that missed one merge: as many as the
    products, where two of them share a column."""
    import torch
    rng = np.random.default_rng(total)
    arows, brows = [], []
    for _ in range(8):
        first = len(brows)
        cols = lo + np.sort(rng.permutation(hi - lo)[:total])
        part = np.split(cols[rng.permutation(total)], np.cumsum(_lengths(total, na))[:-1])
        part[1][0] = part[0][0]                       # two products in one column
        brows += part
        arows.append(np.arange(first, first + na))
    A = _csr(arows, len(brows), rng, dtype)
    B = _csr(brows, hi + 1, rng, dtype)
    import oracle
    right = oracle.row_nnz(A, B)
    assert np.array_equal(right, np.full(8, total - 1))
    da, db = to_dev(A), to_dev(B)
    run_numeric = h._lib.msp_internal_numeric
    run_numeric.argtypes = [ctypes.c_void_p, ctypes.POINTER(binding.c_csr), ctypes.POINTER(binding.c_csr),
                            ctypes.c_void_p, ctypes.POINTER(binding.c_csr_out)]
    for counts, good in [(right, True), (right + 1, False)]:
        n = int(counts.sum())
        cnt = torch.from_numpy(counts.astype(np.int32)).cuda()
        rp = torch.empty(9, dtype=torch.int64, device="cuda")
        col = torch.empty(n, dtype=torch.int32, device="cuda")
        val = torch.empty(n, dtype=da.val.dtype, device="cuda")
        torch.cuda.synchronize()
        out = binding.c_csr_out(8, hi + 1, n, rp.data_ptr(), col.data_ptr(), val.data_ptr(), da.c().dtype)
        assert run_numeric(h._h, ctypes.byref(da.c()), ctypes.byref(db.c()), cnt.data_ptr(), ctypes.byref(out)) == 0
        if good:
            h.sync()
            oracle.compare(rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy(), oracle.spgemm(A, B),
                           TOL[np.dtype(dtype)])
        else:
            with pytest.raises(binding.MspError):
                h.sync()


def _pair(monkeypatch, test, h, *args):
    """The first matrices that an edge case above multiplies."""
    pairs = []
    monkeypatch.setitem(globals(), "check_full", lambda h, A, B, **kw: pairs.append((A, B)))
    test(h, *args)
    return pairs[0]


EDGES = sorted([("row", n) for n in CASES] + [("sort", n) for n in SORT_CASES])


@pytest.mark.parametrize("less", [0, 1])
@pytest.mark.parametrize("kind,name", EDGES)
def test_edges_by_capacity(h, monkeypatch, kind, name, less):
    """The edge cases in rooms of exactly the first row's outputs, or one less
    (rows that do not fit are computed again)."""
    test = test_row_kernel_edges if kind == "row" else test_sort_kernel_edges
    A, B = _pair(monkeypatch, test, h, name, np.float64)
    import oracle
    ref = oracle.spgemm(A, B)
    room = int(ref[0][1]) - less
    pred = binding.Predictor(h, learned.fixed_capacity_params(np.log2(room - 0.5) / 16.0))
    C, _ = h.spgemm_learned(pred, to_dev(A), to_dev(B))
    got = C.to_host()
    oracle.compare(got.row_ptr, got.col, got.val, ref, 1e-12)
    pred.close()


@pytest.mark.parametrize("kind,name,dtype", [(*e, t) for e in EDGES for t in (np.float64, np.float32)]
                         + [("list", n, np.float32) for n in sorted(LIST_CASES)])
def test_edges_in_a_batch(h, monkeypatch, kind, name, dtype):
    """The edge cases as the second problem of a batch, replayed twice."""
    if kind == "list":
        A, B = _pair(monkeypatch, test_list_kernel_edges, h, name)
    else:
        test = test_row_kernel_edges if kind == "row" else test_sort_kernel_edges
        A, B = _pair(monkeypatch, test, h, name, dtype)
    import oracle
    A0 = gen.erdos_renyi(130, 90, 5, seed=91, dtype=dtype)
    B0 = gen.erdos_renyi(90, 500, 4, seed=92, dtype=dtype)
    plan = binding.Batch(h, binding.PackedBatch.from_host([A0, A]), binding.PackedBatch.from_host([B0, B]))
    for _ in range(2):
        plan.execute()
        for p, (x, y) in enumerate([(A0, B0), (A, B)]):
            got = plan.result(p).to_host()
            oracle.compare(got.row_ptr, got.col, got.val, oracle.spgemm(x, y), TOL[np.dtype(dtype)])
    plan.close()


@pytest.mark.parametrize("ncols", [33, 64, 250, 512, 1024])
def test_symbolic_rows_bounded_by_the_width(h, ncols):
    """Rows of at most 64 A entries with more products than columns, in spans
    that start and end anywhere, beside rows of more entries."""
    rng = np.random.default_rng(ncols)
    rows = []
    for _ in range(500):                             # B rows of a stretch of the columns, all of it or single ones
        lo = int(rng.integers(0, ncols))
        hi = int(rng.integers(lo, ncols)) + 1
        n = int(rng.choice([1, hi - lo, (hi - lo + 1) // 2]))
        rows.append(lo + np.sort(rng.permutation(hi - lo)[:n]))
    rows[7] = rows[8] = rows[499] = np.zeros(0, np.int64)
    B = _csr(rows, ncols, rng, np.float64)
    A = gen.erdos_renyi(900, 500, rng.choice([1, 2, 30, 63, 64, 65, 128], size=900), seed=43)
    check_full(h, A, B)
    check_full(h, A, B, tuning=(1, 0, 4096, 1024, -1))
    import oracle
    plan = binding.Batch(h, *[binding.PackedBatch.from_host([x, x]) for x in (A, B)])
    plan.execute()
    got = plan.result(1).to_host()
    oracle.compare(got.row_ptr, got.col, got.val, oracle.spgemm(A, B), 1e-12)
    plan.close()


@pytest.mark.parametrize("rows", [1, 40, 4200])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_global_bin_with_few_and_many_rows(h, rows, dtype):
    """Both shapes of the window kernel and of the symbolic bitmap: rows of some
    19,000 products and 15,000 outputs over 50,000 columns, in several slices."""
    B = gen.erdos_renyi(500, 50_000, 300, seed=71, dtype=dtype)
    A = gen.erdos_renyi(rows, 500, 64, seed=72, dtype=dtype)
    C = run(h, A, B)
    import oracle
    assert np.array_equal(np.diff(C.row_ptr.cpu().numpy()), oracle.row_nnz(A, B))
    check_rows(C, A, B, np.unique(np.linspace(0, rows - 1, 25).astype(int)))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("na", [64, 65, 200])
@pytest.mark.parametrize("total", [8192, 8193, 30_000])
@pytest.mark.parametrize("alone", [True, False])
def test_row_kernel_most_products(h, total, na, alone, dtype):
    """Rows of 257 to 512 outputs on both sides of the products that a wave
    hashes, in one bin (taken in their natural order) and beside others; plain,
    by capacity and in a batch."""
    rng = np.random.default_rng(total + na)
    arows, brows = [], []
    for i in range(40):
        cols = np.sort(rng.permutation(60_000)[:int(rng.integers(300, 500))])
        first = len(brows)
        lens = _lengths(min(total, na * 290) if i % 3 else 700, na)
        brows += [cols[np.sort(rng.permutation(len(cols))[:n])] for n in lens]
        arows.append(np.arange(first, first + na))
        arows.append(np.arange(first, first + (0 if alone else 1 + i % 9)))
    A = _csr(arows, len(brows), rng, dtype)
    B = _csr(brows, 60_000, rng, dtype)
    check_full(h, A, B)
    import oracle
    ref = oracle.spgemm(A, B)
    tol = TOL[np.dtype(dtype)]
    pred = binding.Predictor(h, learned.fixed_capacity_params(np.log2(450) / 16.0))
    got = h.spgemm_learned(pred, to_dev(A), to_dev(B))[0].to_host()
    oracle.compare(got.row_ptr, got.col, got.val, ref, tol)
    pred.close()
    plan = binding.Batch(h, *[binding.PackedBatch.from_host([x]) for x in (A, B)])
    for _ in range(2):
        plan.execute()
        got = plan.result(0).to_host()
        oracle.compare(got.row_ptr, got.col, got.val, ref, tol)
    plan.close()


@pytest.mark.parametrize("rows", [8191, 8192, 20_479, 20_480])
@pytest.mark.parametrize("tuning", [(1, 0, 4096, 1024, 8), (2, 0, 4096, 1024, 8), (1, 1, 4096, 1024, 8),
                                    (2, 2, 4096, 1024, -1)])
def test_many_short_rows_under_every_scale(h, rows, tuning):
    """Both sides of the row counts from which short rows share a wave, alone and
    with longer rows among them, under the tunings that shape their bin."""
    rng = np.random.default_rng(rows)
    B = gen.erdos_renyi(900, 60_000, 7, seed=54)
    A = gen.erdos_renyi(rows, 900, 7, seed=55)
    check_full(h, A, B, tuning=tuning)
    for n in (rows + 900, 66_000 + rows):
        k = np.where(rng.random(n) < 0.03, rng.choice([20, 35, 60] if n < 66_000 else [20, 35], size=n), 7)
        check_full(h, gen.erdos_renyi(n, 900, k, seed=56), B, tuning=tuning)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("room", [40, 100, 200, 400, 900, 1500, 3000])
@pytest.mark.parametrize("na,length", [(700, 12), (60, 150), (300, 60), (2000, 12)])
def test_rooms_far_too_small(h, room, na, length, dtype):
    """Rows of 8000 to 24,000 products in rooms that their outputs fill many times
    over, in every kernel that takes a capacity, beside rows that fit."""
    rng = np.random.default_rng(na + room)
    B = gen.erdos_renyi(4000, 100_000, np.where(np.arange(4000) < 2000, length, 2), seed=73, dtype=dtype)
    rows = [np.sort(rng.permutation(2000)[:na]) if i % 5 == 0 else 2000 + np.sort(rng.permutation(2000)[:18])
            for i in range(200)]
    A = _csr(rows, 4000, rng, dtype)
    import oracle
    pred = binding.Predictor(h, learned.fixed_capacity_params(np.log2(room) / 16.0))
    C, st = h.spgemm_learned(pred, to_dev(A), to_dev(B))
    assert st["overflow_rows"] == 40
    got = C.to_host()
    oracle.compare(got.row_ptr, got.col, got.val, oracle.spgemm(A, B), TOL[np.dtype(dtype)])
    pred.close()
