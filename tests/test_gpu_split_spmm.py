"""fp32 SpMM of dense sparse matrices on the fp16 matrix cores (two terms per number), against the oracle.  Tolerance: a result is four
chains, each of the products of high terms for every sixteen of a quarter of A's columns, added to the sum with no more than four
roundings of 2^-23 at most, and of three smaller products in a sum of their own, 2^-11 of that; the terms hold each of two numbers to 2^-23 of it:
(16 (k / 64 + 1) + 16) 2^-24 of the sum of absolute products, twice what this comes to.  That bound holds for any signs and is far above what normally
distributed inputs give, for which the 2-norm of the error has to be no larger than that of a chain of fp32 multiply-adds over the row's entries, the
sums before."""
import ctypes

import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_slab_pieces import odd_csr


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


def runs_split(m, k, n, nnz):
    import paper_2006_10901_amd as spdl
    s = spdl.spdl_select_spmm(m, k, n, nnz, 4, 0, 0)
    form = ctypes.CDLL(spdl.LIB_PATH).spdl_debug_slab_form(m, k, n, nnz)
    return spdl.spdl_variant_name(0, s["variant"]) == "slabdma" and form == 4 and (s["rows_per_block"], s["block_threads"], s["grid_y"]) == (64, 1024, 1)


def test_where_dense_matrices_are_multiplied_whole():
    assert runs_split(8192, 10240, 128, int(8192 * 10240 * 0.3)) and not runs_split(8192, 10240, 128, int(8192 * 10240 * 0.15))
    assert runs_split(6765, 2169, 120, int(6765 * 2169 * 0.28)) and runs_split(4096, 1024, 1024, int(4096 * 1024 * 0.3))
    assert not runs_split(4096, 1024, 4096, int(4096 * 1024 * 0.3))       # wide outputs
    assert not runs_split(8192, 799, 128, int(8192 * 799 * 0.5))          # few columns
    assert not runs_split(4096, 4096, 128, int(4096 * 4096 * 0.4))        # 128 tiles: rows shared
    assert not runs_split(8192, 10240, 32, int(8192 * 10240 * 0.4))       # half a tile


def spmm(g, A, n, B, order=None, bias=None):
    """The arrays of A, B and C at odd element addresses with NaN and far columns around."""
    import torch
    import paper_2006_10901_amd as spdl
    assert runs_split(A.m, A.k, n, A.nnz)
    d = g.DevCsr(A)
    ci = torch.full((A.nnz + 2,), 1 << 30, dtype=torch.int32, device="cuda")
    val, b, c = (torch.full((size + 2,), float("nan"), device="cuda") for size in (A.nnz, A.k * n, A.m * n))
    ci[1:-1], val[1:-1], b[1:-1] = d.ci, d.val, g.dev(B).view(-1)
    C = c[1:-1].view(A.m, n)
    args = (A.m, A.k, n, A.nnz, d.ro, ci[1:-1], val[1:-1], g.dev(order) if order is not None else None, b[1:-1].view(A.k, n))
    spdl.spdl_spmm(*args, C) if bias is None else spdl.spdl_spmm_bias_relu(*args, g.dev(bias), True, C)
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    assert np.isnan(got[0]) and np.isnan(got[-1])
    return got[1:-1].reshape(A.m, n)


def tolerance(k):
    return (16 * (k // 64 + 1) + 16) * 2.0 ** -24


def chain(A, B, rows):
    """The rows' results as chains of fp32 multiply-adds in stored order (products are exact in 64 bits)."""
    acc = np.zeros((len(rows), B.shape[1]), np.float32)
    first, last = A.row_offsets[rows], A.row_offsets[rows + 1]
    for t in range(int(np.max(last - first, initial=0))):
        on = np.flatnonzero(first + t < last)
        p = first[on] + t
        acc[on] = (A.values[p].astype(np.float64)[:, None] * B[A.column_indices[p]] + acc[on]).astype(np.float32)
    return acc


def assert_as_exact_as_a_chain(got, ref, A, B, rows):
    ours, theirs = np.linalg.norm(got[rows] - ref[rows]), np.linalg.norm(chain(A, B, rows) - ref[rows])
    assert ours <= theirs, (ours / theirs, theirs / np.linalg.norm(ref[rows]))


# (rows around whole panels; columns around whole stages of 128 and sixteens, and fewer than a quarter of a stage over; columns of C around whole
# tiles, halves and fours; two, three and four sixteens of look-ahead and rows beyond; eight groups of tiles and up to 2048 rows)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,density", [(8256, 1039, 65, 0.3), (8200, 816, 33, 0.5), (4161, 896, 130, 0.3), (4100, 1030, 127, 0.7), (4159, 801, 189, 0.9),
                                           (1000, 1025, 700, 0.4), (2049, 1153, 322, 0.33), (8197, 1001, 64, 0.25), (1100, 1552, 512, 0.22)])
def test_split_spmm(g, oracle_lib, m, k, n, density):
    A = odd_csr(m, k, density, 7500 + m)
    B = wl.dense(k, n, 7501 + n)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B, oracle_lib.row_order(m, A.row_offsets))
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - ref) <= tolerance(k) * S)
    assert_as_exact_as_a_chain(got, ref, A, B, np.flatnonzero(np.diff(A.row_offsets) > 150)[:300])
    assert np.array_equal(spmm(g, A, n, B), got)
    bias = np.random.default_rng(7502).standard_normal(m).astype(np.float32)
    ref, S = oracle_lib.spmm_bias_relu(m, k, n, A.row_offsets, A.column_indices, A.values, B, bias, True)
    assert np.all(np.abs(spmm(g, A, n, B, None, bias) - ref) <= tolerance(k) * (S + np.abs(bias)[:, None]))


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1025, 2169])
def test_split_spmm_is_as_exact_as_a_chain_for_rows_of_any_length(g, oracle_lib, k):
    """Rows of few entries between long ones, each length by itself; and rows of many zeros with one number, whose product has to come out to
    what the terms of two numbers leave out (2^-23 each) and three roundings: every one of the four products of terms counts there."""
    m, n, least = 4161, 130, 72 + k // 24
    lengths = [1, 2, 3, 16, 17, 31, 32, 33, 49, least - 1, least, least + 20, 2 * least]
    rng = np.random.default_rng(7300 + k)
    lens = np.full(m, int(0.7 * k))
    lens[::2] = np.resize(lengths, len(lens[::2]))
    cols = np.concatenate([np.sort(rng.permutation(k)[:x]) for x in lens]).astype(np.int32)
    A = wl.Csr(m, k, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), cols, rng.standard_normal(int(lens.sum())).astype(np.float32))
    single = np.arange(1, m, 8)
    for i in single:
        row = A.values[A.row_offsets[i]:A.row_offsets[i + 1]]
        row[rng.permutation(len(row))[1:]] = 0
    B = rng.standard_normal((k, n)).astype(np.float32)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B)
    for x in lengths:
        assert_as_exact_as_a_chain(got, ref, A, B, np.flatnonzero(lens == x))
    assert np.all(np.abs(got[single] - ref[single]) <= 7 * 2.0 ** -24 * S[single])


@pytest.mark.gpu
def test_split_spmm_of_rows_in_no_order(g, oracle_lib):
    """Rows of ascending runs, exchanged, and columns stored twice, next to each other and not: every way in which the cursor can be misled."""
    m, k, n = 4161, 1025, 130
    A = odd_csr(m, k, 0.35, 7600)
    rng = np.random.default_rng(7601)
    for i in range(m):
        row = A.column_indices[A.row_offsets[i]:A.row_offsets[i + 1]]
        if len(row) < 100:
            continue
        if i % 4 == 1:
            runs = np.split(row.copy(), np.sort(rng.integers(0, len(row), int(rng.integers(2, 8)))))
            row[:] = np.concatenate([runs[j] for j in rng.permutation(len(runs))])
        elif i % 4 == 2:
            at = int(rng.integers(0, len(row) - 40))
            row[at + int(rng.integers(1, 40))] = row[at]
        elif i % 4 == 3 and i % 8 == 3:
            at = int(rng.integers(0, len(row) - 1))
            row[at], row[at + 1] = row[at + 1], row[at]
    B = wl.dense(k, n, 7602)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B)
    longest = int(np.max(np.diff(A.row_offsets)))                     # (gathered: a chain of the row's entries)
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - ref) <= max(tolerance(k), (longest + 8) * 2.0 ** -24) * S)


@pytest.mark.gpu
@pytest.mark.parametrize("density", [0.6, 0.5])                       # four and three sixteens of look-ahead
def test_split_spmm_of_rows_whose_middle_lies_in_a_later_stage(g, oracle_lib, density):
    """Four adjacent rows, one of which takes another round of its first stage, and a sixteen of which no row has an entry in the stage with
    entries of the stage behind it."""
    m, k, n = 4161, 1025, 130
    A = odd_csr(m, k, density, 7650)
    rows = np.split(A.column_indices, A.row_offsets[1:-1])
    run, far = lambda first, count: np.arange(first, first + count), np.arange(300, 316)
    patterns = [[[run(0, 16), far, run(20, 40)], [], [], [run(0, 16), far, run(100, 16)]],
                [[run(0, 16), far, run(20, 70)], [], [run(0, 16), far, run(100, 16)], [run(0, 16), far, far + 16, run(90, 16)]],
                [[run(0, 16), run(20, 40)], [run(0, 16), far, run(100, 16)], [], [run(0, 32), far, run(100, 16)]]]
    for i in range(0, m - 8, 8):
        for j, parts in enumerate(patterns[i // 8 % 3]):
            rows[i + j] = np.concatenate(parts).astype(np.int32) if parts else np.zeros(0, np.int32)
    lens = np.array([len(r) for r in rows])
    values = np.random.default_rng(7651).standard_normal(lens.sum()).astype(np.float32)
    A = wl.Csr(m, k, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.concatenate(rows), values)
    B = wl.dense(k, n, 7652)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B)
    assert np.all(np.abs(got - ref) <= max(tolerance(k), (int(lens.max()) + 8) * 2.0 ** -24) * S)


@pytest.mark.gpu
def test_split_spmm_keeps_non_finite_values_and_the_whole_range(g, oracle_lib):
    """Infinities and NaN reach the results that depend on them and no others, though zeros are multiplied; numbers at either end of the
    range, whose scaled sums need not be finite, cost time, not bits."""
    m, k, n = 4161, 1025, 130
    A = odd_csr(m, k, 0.35, 7700)
    B = wl.dense(k, n, 7701)
    values = A.values
    for scale_a, scale_b in ((2.0 ** -100, 2.0 ** -20), (2.0 ** -126, 1.0), (2.0 ** -126, 2.0 ** 100), (2.0 ** 105, 2.0 ** -90), (2.0 ** 60, 2.0 ** 50)):
        A.values, b = (values * np.float32(scale_a)).astype(np.float32), (B * np.float32(scale_b)).astype(np.float32)
        ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, b)
        # (a denormal product or sum is a multiple of 2^-149)
        assert np.all(np.abs(spmm(g, A, n, b) - ref) <= max(tolerance(k), (k + 8) * 2.0 ** -24) * S + k * 2.0 ** -149), (scale_a, scale_b)
    A.values = values.copy()
    B[5, 0], B[700, 64], B[k - 1, n - 1], B[300, 33] = np.inf, np.nan, -np.inf, np.float32(3e38)
    A.values[A.row_offsets[200] + 3], A.values[A.row_offsets[3000]] = np.inf, np.nan
    with np.errstate(invalid="ignore", over="ignore"):
        ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B).astype(np.float64)
    inside = np.abs(ref) < 1e38
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and 0 < np.count_nonzero(~inside) < m * n // 20
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.all(np.abs(got[inside] - ref[inside]) <= max(tolerance(k), (k + 8) * 2.0 ** -24) * S[inside])


@pytest.mark.gpu
@pytest.mark.parametrize("bad_rows", [1, 2, 3, 5, 33, 64])            # of each panel of 64
@pytest.mark.parametrize("bad_columns", [(), (7,), (0, 66, 129), (1, 21, 45, 62, 128)])
def test_split_spmm_shares_out_what_is_gathered(g, oracle_lib, bad_rows, bad_columns):
    """Few and many rows that have to be gathered (one column stored twice, or a NaN) and few and many fours of columns (an infinity in B): rows, fours
    and parts of a row for every power of two of threads, rows of 0, 1, 16, 17 and all entries among them."""
    m, k, n = 4161, 1025, 130
    A = odd_csr(m, k, 0.35, 7800)
    rows = [r.copy() for r in np.split(A.column_indices, A.row_offsets[1:-1])]
    for i, r in enumerate(rows):
        if i % 64 % 29 == 11:
            rows[i] = np.arange((0, 1, 16, 17, k)[i // 64 % 5], dtype=np.int32)
    lens = np.array([len(r) for r in rows])
    A = wl.Csr(m, k, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.concatenate(rows),
               np.random.default_rng(7801).standard_normal(lens.sum()).astype(np.float32))
    for i in range(m):
        at, end = A.row_offsets[i], A.row_offsets[i + 1]
        if (i % 64) * 37 % 64 < bad_rows and end - at > 1:
            if i % 3 == 0:
                A.values[end - 1] = np.nan
            else:
                A.column_indices[at + (end - at) // 2] = A.column_indices[at + (end - at) // 2 - 1]
    B = wl.dense(k, n, 7802)
    for c in bad_columns:
        B[(c * 31 + 400) % k, c] = np.inf if c % 2 else -np.inf
    with np.errstate(invalid="ignore"):
        ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = spmm(g, A, n, B).astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    inside = np.isfinite(ref)
    assert np.all(np.abs(got[inside] - ref[inside]) <= max(tolerance(k), (k + 8) * 2.0 ** -24) * S[inside])


@pytest.mark.gpu
def test_split_spmm_gathers_no_slower_than_this(g):
    """What an infinity in every result costs: 4.8 times the whole time where it was measured, 21 times with each result left to the thread that has
    it."""
    import torch
    import paper_2006_10901_amd as spdl
    m, k, n = 8192, 4096, 128
    A = wl.uniform_mask_csr(m, k, 0.3, 7900)
    assert runs_split(m, k, n, A.nnz)
    d, C = g.DevCsr(A), torch.empty((m, n), device="cuda")
    B = wl.dense(k, n, 7901)
    bad = B.copy()
    bad[k // 2] = np.inf
    times = []
    for b in (g.dev(B), g.dev(bad)):
        runs = []
        for _ in range(7):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(5):
                spdl.spdl_spmm(m, k, n, A.nnz, d.ro, d.ci, d.val, None, b, C)
            end.record()
            end.synchronize()
            runs.append(start.elapsed_time(end))
        times.append(min(runs))
    assert times[1] < 9 * times[0], times
