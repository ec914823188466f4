"""fp32 SpMM of dense sparse matrices on the matrix cores (two fp16 terms per number), with numbers of every magnitude: each row of A and each column
of B is taken times a power of two that falls when a larger number comes.  Tolerance: the bound for four products of terms, as many roundings as
the sum has steps of sixteen columns, and 8 sqrt(k) for the bits that the common powers of two may cost a sum:
(16 (k / 64 + 1) + 16 + 8 sqrt(k)) 2^-24 of the sum of the absolute products of A's stored entries, whatever else the row, the column or the rows of B
hold that A does not store.  That is for any signs; over all results the root of the mean square is no more than half of sqrt(k) 2^-24, what
roundings of as many terms come to, so that no part of them may be far off."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_slab_pieces import odd_csr
from tests.test_gpu_split_spmm import runs_split


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


def numbers(kind, A, n):
    rng = np.random.default_rng(8100)
    B = rng.standard_normal((A.k, n)).astype(np.float32)
    rows = np.repeat(np.arange(A.m), np.diff(A.row_offsets))
    at, v = A.column_indices / A.k, A.values
    if kind == "rows and columns":
        v *= np.exp2(rng.integers(-40, 41, A.m))[rows].astype(np.float32)
        B *= np.exp2(rng.integers(-40, 41, n)).astype(np.float32)
    elif kind == "growing":                                # a new power of two every few stages, of single rows and of all
        v *= np.exp2(np.floor(np.where(rows % 3 == 0, 40, np.where(rows % 3 == 1, 12, 0)) * at)).astype(np.float32)
        B *= np.exp2(np.floor(30 * np.arange(A.k) / A.k))[:, None].astype(np.float32)
    elif kind == "falling":
        v *= np.exp2(-np.floor(20 * at)).astype(np.float32)
        B *= np.exp2(-np.floor(20 * np.arange(A.k) / A.k))[:, None].astype(np.float32)
    elif kind == "zeros first":
        v[at < 0.4] = 0
        B[:A.k // 3] = 0
        v[rows % 5 == 0] = 0
        B[:, ::7] = 0
    elif kind == "spikes":                                 # also in a stage's second round of sixteens
        v[rng.integers(0, len(v), A.m)] *= np.float32(2.0 ** 40)
        B[rng.integers(0, A.k, n), np.arange(n)] *= np.float32(2.0 ** 30)
    elif kind == "tiny":
        v *= np.float32(2.0 ** -120)
        B *= np.float32(2.0 ** 30)
    elif kind == "huge":
        v *= np.float32(2.0 ** -60)
        B *= np.float32(2.0 ** 120)
    elif kind == "few in a column":                        # sums of nothing, and of a few entries of a row
        B[:, 3:9] = 0
        B[5, 3], B[A.k // 2, 4], B[::97, 5] = 1.5, -0.7, 1.0
    return B


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "rows and columns", "growing", "falling", "zeros first", "spikes", "tiny", "huge", "few in a column"])
@pytest.mark.parametrize("m,k,n,density", [(4161, 1025, 130, 0.25), (2100, 1300, 331, 0.45)])
def test_split_spmm_of_any_magnitude(g, oracle_lib, kind, m, k, n, density):
    A = odd_csr(m, k, density, 8101 + k)
    B = numbers(kind, A, n)
    assert runs_split(m, k, n, A.nnz)
    check(g, oracle_lib, A, B, n)


def check(g, oracle_lib, A, B, n):
    ref, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    got = g.gpu_spmm(A, B, n)
    assert np.all(np.isfinite(got))
    off = np.abs(got - ref) - 2.0 ** -149
    assert np.all(off <= (16 * (A.k // 64 + 1) + 16 + 8 * np.sqrt(A.k)) * 2.0 ** -24 * S)
    part = np.maximum(off, 0)[S > 0] / S[S > 0]
    assert np.sqrt(np.mean(part ** 2)) <= np.sqrt(A.k) * 2.0 ** -25


@pytest.mark.gpu
@pytest.mark.parametrize("large", [2.0 ** 20, 2.0 ** 30, 2.0 ** 40, 1e15, 1e20, 1e30])
@pytest.mark.parametrize("where", ["B", "A", "both"])
def test_large_numbers_reach_only_the_sums_that_they_are_in(g, oracle_lib, where, large):
    """Finite numbers far above all others, early, in the middle and last: in rows of B that most rows of A do not store, and in entries of A
    whose row of B has zeros; where A stores them and B has none, they are the sum's."""
    m, k, n = 4161, 1025, 130
    A = odd_csr(m, k, 0.25, 8200)
    B = numbers("plain", A, n)
    assert runs_split(m, k, n, A.nnz)
    for i, t in enumerate([1, 300, 517, 800, 1024]):
        if where != "A":
            B[t, i::7] = np.float32(large) * B[t, i::7]
        if where != "B":
            A.values[A.column_indices == (t + 11) % k] *= np.float32(large)
            B[(t + 11) % k, i % 3::3] = 0
    check(g, oracle_lib, A, B, n)


@pytest.mark.gpu
@pytest.mark.parametrize("row", [1, 12, 20, 30, 40, 127, 300, 517, 1024])
def test_a_larger_number_leaves_the_columns_beside_it_alone(g, row):
    """In whichever half of a sixteen it lies, its column of B gets another power of two and is multiplied like any other: the results of the columns
    that would be gathered with it keep their bits.  (A hundredth of the rows may have a sum that is small enough to be gathered.)"""
    m, k, n = 4161, 1025, 130
    A = wl.uniform_mask_csr(m, k, 0.25, 8300)
    B = wl.dense(k, n, 8301)
    assert runs_split(m, k, n, A.nnz)
    before = g.gpu_spmm(A, B, n)
    B[row, 7] = 200.0
    B[row, 37] = -300.0
    after = g.gpu_spmm(A, B, n)
    others = np.setdiff1d(np.arange(n), [7, 37])
    assert np.count_nonzero(np.any(before[:, others] != after[:, others], axis=1)) <= m // 100


def time_of(spdl, A, d, B, n):
    """Milliseconds of five calls, the least of seven."""
    import torch
    C, runs = torch.empty((A.m, n), device="cuda"), []
    for _ in range(7):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(5):
            spdl.spdl_spmm(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, None, B, C)
        end.record()
        end.synchronize()
        runs.append(start.elapsed_time(end))
    return min(runs)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["ones", "one in a thousand"])
def test_sums_that_are_small_and_right_cost_little(g, kind):
    """A and B of plus and minus ones, where one sum in a hundred is zero, and one number in a thousand of B that is not zero, where one sum in three
    is.  Measured: 1.2 and 1.4 times the time of normally distributed numbers; 4.1 and 5.1 times it where all of them are gathered, by rows."""
    import paper_2006_10901_amd as spdl
    m, k, n = 8192, 4096, 128
    A = wl.uniform_mask_csr(m, k, 0.3, 8400)
    B = wl.dense(k, n, 8401)
    assert runs_split(m, k, n, A.nnz)
    plain = time_of(spdl, A, g.DevCsr(A), g.dev(B), n)
    if kind == "ones":
        A.values, B = np.sign(A.values), np.sign(B)
    else:
        B[np.random.default_rng(8402).random((k, n)) >= 0.001] = 0
    small = time_of(spdl, A, g.DevCsr(A), g.dev(B), n)
    print(f"{small / plain:.2f} times {plain / 5:.4f} ms")
    assert small < 2 * plain, (plain, small)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [127, 130, 189])                         # (a last four of three and two columns and of one)
@pytest.mark.parametrize("tiny", [0, 1, 40])
def test_small_sums_of_numbers_that_lose_nothing_and_of_some_that_do(g, oracle_lib, tiny, n):
    """Numbers of -1, 0 and 1, of which whole tiles have sums of nothing or of a few: exact.  Then with a few numbers, in A and in B, that are far below
    the others: what they are all of a sum is as good as any other."""
    m, k = 4161, 1025
    A = odd_csr(m, k, 0.25, 8500)
    rng = np.random.default_rng(8501)
    A.values = rng.integers(-1, 2, A.nnz).astype(np.float32)
    B = rng.integers(-1, 2, (k, n)).astype(np.float32)
    B[rng.random((k, n)) < 0.6] = 0
    B[:, ::5] = 0
    B[17, ::10] = 1
    B[:, 64:72] *= np.float32(2.0 ** -120)                             # (a column of nothing else)
    for i in range(tiny):
        B[rng.integers(0, k, 8), rng.integers(0, n, 8)] = np.float32(2.0 ** -30) * rng.standard_normal(8)
        A.values[rng.integers(0, A.nnz, 8)] = np.float32(2.0 ** -30) * rng.standard_normal(8)
    assert runs_split(m, k, n, A.nnz)
    if tiny:
        check(g, oracle_lib, A, B, n)
        return
    ref, _ = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    assert np.array_equal(g.gpu_spmm(A, B, n), ref.astype(np.float32))
