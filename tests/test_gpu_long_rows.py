"""Row-splitting SpMM with a wave per row: rows of more than twice the mean length (at least 64 entries) are
walked by the four waves of a workgroup, in fp32 from a mean of 96 entries on, or of 16 where the caller says that rows are unequal, and in half precision with few waves every row is.  Against the oracle; tolerance: a chain of at most as many
multiply-adds as the longest row has entries and three additions, (r + 3) 2^-24 of the sum of absolute products, in half precision rounded once
more."""
import numpy as np
import pytest

import workloads as wl


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


@pytest.fixture
def force():
    import paper_2006_10901_amd as spdl
    yield spdl.spdl_force_variant
    spdl.spdl_force_variant(0, -1)


def rows_csr(k, lens, seed):
    rng = np.random.default_rng(seed)
    ro = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(k, size=l, replace=False)) for l in lens] + [np.zeros(0, int)]).astype(np.int32)
    return wl.Csr(len(lens), k, ro, ci, rng.standard_normal(len(ci)).astype(np.float16))


def test_when_a_workgroup_has_one_row(force):
    import paper_2006_10901_amd as spdl
    force(0, 0)
    rows = lambda m, n, avg, eb=2: spdl.spdl_select_spmm(m, 900, n, m * avg, eb, 0, 0)["rows_per_block"]
    assert rows(799, 512, 16) == 1 and rows(799, 512, 15) == 4 and rows(800, 512, 49) == 4 and rows(800, 512, 50) == 1
    assert rows(1599, 400, 50) == 1 and rows(1600, 400, 300) == 4 and rows(799, 1024, 50) == 1 and rows(800, 1024, 50) == 4
    assert rows(300, 511, 100) == 4 and rows(300, 400, 100, 4) == 4


# 97 and 1601 rows: the last workgroup is incomplete.  Mean lengths from 24 to 34 put the line at 64 .. 68 entries, in fp32 from 100 to 120 at 200 .. 240:
# rows on both sides of it, empty ones, one of every column, and two to four long ones among the rows of one workgroup (i, i + 25, i + 50, i + 75 of 97)
@pytest.mark.gpu
@pytest.mark.parametrize("n,dtype", [(n, np.float16) for n in (257, 263, 400, 511, 513, 516, 1000, 2049)] + [(n, np.float32) for n in (257, 260, 515, 1024)])
@pytest.mark.parametrize("m", [97, 1601])
def test_long_rows(g, oracle_lib, force, m, n, dtype):
    import torch
    import paper_2006_10901_amd as spdl
    f16, k = dtype == np.float16, 300
    rng = np.random.default_rng(9000 + m)
    lens = rng.integers(0, 48, m) if f16 else rng.integers(80, 130, m)
    grid = -(-m // 4)
    for at, long in ((0, (300, 0, 65, 63)), (5, (64, 65, 66, 67)), (7, (200, 180, 1, 210)), (grid - 1, (80, 90, 100, 0))) + (() if f16 else ((8, (199, 241, 260, 300)),)):
        for w, l in enumerate(long):
            if w * grid + at < m:
                lens[w * grid + at] = l
    if f16:
        lens[1::7] = np.maximum(lens[1::7], 40)
    A = rows_csr(k, lens, 9001 + m)
    A.values = A.values.astype(dtype)
    assert 24 <= A.nnz // m < 40 if f16 else 96 <= A.nnz // m < 120
    force(0, 0)
    s = spdl.spdl_select_spmm(m, k, n, A.nnz, 2 if f16 else 4, 0, 0)
    assert spdl.spdl_variant_name(0, s["variant"]) == "rowsplit" and s["lanes_per_row"] == 64 and (f16 or s["rows_per_block"] == 4)
    B = wl.dense(k, n, 9002 + n, dtype)
    bias = rng.standard_normal(m).astype(dtype)
    d = g.DevCsr(A)
    b, c = (torch.full((size + 2,), float("nan"), dtype=torch.float16 if f16 else torch.float32, device="cuda") for size in (k * n, m * n))
    b[1:-1] = g.dev(B).view(-1)
    ref, S = oracle_lib.spmm_bias_relu(m, k, n, A.row_offsets, A.column_indices, A.values.astype(np.float32), B.astype(np.float32), bias.astype(np.float32), True)
    S = S + np.abs(bias.astype(np.float64))[:, None]
    bound = (int(lens.max()) + 3) * 2.0 ** -24 * S + (2.0 ** -11 * np.abs(ref) + 2.0 ** -25 if f16 else 0.0)
    bits = []
    for order in (None, oracle_lib.row_order(m, A.row_offsets), rng.permutation(m).astype(np.int32)):
        c[1:-1] = float("nan")
        (spdl.spdl_spmm_bias_relu_f16 if f16 else spdl.spdl_spmm_bias_relu)(m, k, n, A.nnz, d.ro, d.ci, d.val, None if order is None else g.dev(order), b[1:-1].view(k, n), g.dev(bias), True,
                                     c[1:-1].view(m, n))
        torch.cuda.synchronize()
        got = c.cpu().numpy()
        assert np.isnan(got[0]) and np.isnan(got[-1]) and np.all(np.isfinite(got[1:-1]))
        assert np.all(np.abs(got[1:-1].reshape(m, n).astype(np.float64) - ref) <= bound)
        bits.append(got[1:-1])
    assert np.array_equal(bits[0], bits[1]) and np.array_equal(bits[0], bits[2])        # the order of the rows moves work, not bits


# (means of 19 .. 38: the line at 64 .. 76 entries.  The call that says nothing about the rows walks each by one wave there, in one chain: which rows
# are shared shows in the last bits.)
@pytest.mark.gpu
@pytest.mark.parametrize("n", [257, 260, 515, 1024])
@pytest.mark.parametrize("m,least", [(97, 0), (97, 16), (1601, 0), (1601, 8)])
def test_long_rows_of_a_caller_who_knows_them(g, oracle_lib, force, m, least, n):
    import torch
    import paper_2006_10901_amd as spdl
    k = 300
    rng = np.random.default_rng(9100 + m)
    lens = rng.integers(least, 40, m)
    grid = -(-m // 4)
    for at, long in ((0, (300, 0, 71, 63)), (5, (64, 65, 66, 67)), (7, (200, 180, 1, 210)), (grid - 1, (80, 90, 100, 0))):
        for w, l in enumerate(long):
            if w * grid + at < m:
                lens[w * grid + at] = l
    A = rows_csr(k, lens, 9101 + m)
    A.values = A.values.astype(np.float32)
    mean = A.nnz // m
    assert 16 <= mean < 40
    force(0, 0)
    s = spdl.spdl_select_spmm(m, k, n, A.nnz, 4, 0, 0)
    assert spdl.spdl_variant_name(0, s["variant"]) == "rowsplit" and (s["lanes_per_row"], s["rows_per_block"]) == (64, 4)
    B = wl.dense(k, n, 9102 + n)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    d = g.DevCsr(A)
    b = torch.full((k * n + 2,), float("nan"), device="cuda")
    b[1:-1] = g.dev(B).view(-1)
    plain, c = torch.empty((m, n), device="cuda"), torch.full((m * n + 2,), float("nan"), device="cuda")
    spdl.spdl_spmm(m, k, n, A.nnz, d.ro, d.ci, d.val, None, b[1:-1].view(k, n), plain)
    spdl.spdl_spmm_skewed(m, k, n, A.nnz, d.ro, d.ci, d.val, b[1:-1].view(k, n), c[1:-1].view(m, n))
    torch.cuda.synchronize()
    got = c.cpu().numpy()
    assert np.isnan(got[0]) and np.isnan(got[-1])
    got = got[1:-1].reshape(m, n)
    assert np.all(np.abs(got - ref) <= (int(lens.max()) + 3) * 2.0 ** -24 * S)
    moved = np.any(got != plain.cpu().numpy(), axis=1)
    shared = lens > max(64, 2 * mean)
    assert np.all(moved[lens >= 80]) and not np.any(moved[~shared]) and np.count_nonzero(shared) >= 5


# (a wave per row, rows shared by four, and a row to a workgroup: the same products and sums by either kind of index)
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,rows", [(97, 257, 4), (97, 516, 1), (799, 512, 1), (1601, 400, 4), (1601, 2049, 4)])
def test_long_rows_by_indices_of_two_bytes(g, oracle_lib, force, m, n, rows):
    import torch
    import paper_2006_10901_amd as spdl
    k = 300
    rng = np.random.default_rng(9200 + m)
    lens = rng.integers(16, 48, m)
    lens[::9] = rng.integers(60, 300, len(lens[::9]))
    A = rows_csr(k, lens, 9201 + m)
    assert A.nnz // m >= 24
    force(0, 0)
    s = spdl.spdl_select_spmm(m, k, n, A.nnz, 2, 0, 0)
    assert spdl.spdl_variant_name(0, s["variant"]) == "rowsplit" and (s["lanes_per_row"], s["rows_per_block"]) == (64, rows)
    B = wl.dense(k, n, 9202 + n, np.float16)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values.astype(np.float32), B.astype(np.float32))
    d, b = g.DevCsr(A), g.dev(B)
    c4, c2 = (torch.full((m, n), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
    order = g.dev(oracle_lib.row_order(m, A.row_offsets))
    spdl.spdl_spmm_f16(m, k, n, A.nnz, d.ro, d.ci, d.val, order, b, c4)
    spdl.spdl_spmm_f16_i16(m, k, n, A.nnz, d.ro, d.ci.to(torch.int16), d.val, order, b, c2)
    torch.cuda.synchronize()
    got = c2.cpu().numpy()
    assert np.array_equal(got, c4.cpu().numpy())
    assert np.all(np.abs(got - ref) <= (int(lens.max()) + 3) * 2.0 ** -24 * S + 2.0 ** -11 * np.abs(ref) + 2.0 ** -25)
