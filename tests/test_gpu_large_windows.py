"""The window kernels with sixteen waves to a workgroup and a window of 576 rows, which callers who say that the entries form a band get where their
rounds of workgroups are filled: on bands, on masks that are none, on rows in no order and on rows that are shared among the waves, against the
oracle.  Tolerance: a result is a chain of fp32 multiply-adds over four to sixteen parts of a row (of the dot product), (length + 16) 2^-24 of the sum
of absolute products."""
import numpy as np
import pytest

import workloads as wl


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


def mask(m, k, band, scattered, seed, shift=0):
    """`band` columns around the diagonal and some `scattered` ones per row, which lie the more densely the nearer."""
    rng = np.random.default_rng(seed)
    rows = []
    for i in range(m):
        centre = min(max(i * k // m + shift, 0), k - 1)
        far = centre + rng.choice([-1, 1], scattered) * (band // 2 + np.exp(rng.uniform(0, np.log(k), scattered)).astype(int))
        cols = np.concatenate([np.arange(centre - band // 2, centre + band // 2 + 1), far])
        rows.append(np.unique(cols[(cols >= 0) & (cols < k)]))
    return rows


def csr(m, k, rows, seed):
    ro = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return wl.Csr(m, k, ro, np.concatenate(rows).astype(np.int32), np.random.default_rng(seed).standard_normal(int(ro[-1])).astype(np.float32))


def check(g, oracle_lib, A, n, sddmm=True):
    import torch
    import paper_2006_10901_amd as spdl
    rng = np.random.default_rng(9000 + n)
    d = g.DevCsr(A)
    longest = int(np.max(np.diff(A.row_offsets)))
    B = rng.standard_normal((A.k, n)).astype(np.float32)
    C = torch.full((A.m, n), float("nan"), device="cuda")
    spdl.spdl_spmm_banded(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, g.dev(B), C)
    ref, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    got = C.cpu().numpy()
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - ref) <= (longest + 16) * 2.0 ** -24 * S)
    if not sddmm:
        return
    L, out = rng.standard_normal((A.m, n)).astype(np.float32), torch.full((A.nnz,), float("nan"), device="cuda")
    spdl.spdl_sddmm_banded(A.m, A.k, n, A.nnz, d.ro, d.ci, g.dev(L), g.dev(B), out)
    ref, S = oracle_lib.sddmm(A.m, A.k, n, A.row_offsets, A.column_indices, L, B)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - ref) <= (n + 16) * 2.0 ** -24 * S)


# (SpMM with sixteen waves: 154 .. 256 workgroups of 16 rows and tile of 64 columns, or as many over whole rounds; SDDMM 2560 .. 4096 rows)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n,band", [(4096, 4096, 64, 257), (2560, 2560, 33, 600), (2559, 2559, 64, 601), (4095, 3000, 36, 33), (4081, 5000, 50, 575),
                                        (1281, 1281, 100, 129), (2033, 577, 128, 65), (2700, 576, 64, 257), (2600, 100, 64, 41), (8190, 4100, 65, 257)])
def test_bands(g, oracle_lib, m, k, n, band):
    check(g, oracle_lib, csr(m, k, mask(m, k, band, 40, 9100 + m), 9101), n)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 100])
def test_rows_that_are_no_band(g, oracle_lib, n):
    m = k = 2700 if n == 64 else 3500
    rng = np.random.default_rng(9200)
    rows = [np.sort(rng.permutation(k)[:int(rng.integers(0, 300))]) for _ in range(m)]
    for i in range(0, m, 16):                                # empty first rows of workgroups
        rows[i] = rows[i][:0]
    check(g, oracle_lib, csr(m, k, rows, 9201), n)
    for i in range(m):                                       # in no order, with columns stored twice
        rows[i] = rng.permutation(np.concatenate([rows[i], rows[i][:5]]))
    check(g, oracle_lib, csr(m, k, rows, 9202), n)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 128])
def test_rows_shared_among_sixteen_waves(g, oracle_lib, n):
    m, k = 2700 if n == 64 else 1400, 3000
    rows = mask(m, k, 65, 20, 9300)
    rng = np.random.default_rng(9301)
    for i in (0, 15, 16, 17, 700, 701, m - 1):
        rows[i] = np.sort(rng.permutation(k)[:int(rng.integers(600, k))])
    check(g, oracle_lib, csr(m, k, rows, 9302), n)


@pytest.mark.gpu
def test_what_lies_outside_a_row_does_not_reach_it(g):
    """Infinities and NaN in rows of B that a sparse row does not name, inside its window and outside."""
    import torch
    import paper_2006_10901_amd as spdl
    m = k = 2700
    n = 64
    rows = [r[(r % 7 != 3)] for r in mask(m, k, 257, 40, 9400)]
    A = csr(m, k, rows, 9401)
    rng = np.random.default_rng(9402)
    B = rng.standard_normal((k, n)).astype(np.float32)
    bad = B.copy()
    bad[3::14], bad[10::14] = np.inf, np.nan
    d = g.DevCsr(A)
    results = []
    for b in (B, bad):
        C, out = torch.empty((m, n), device="cuda"), torch.empty(A.nnz, device="cuda")
        spdl.spdl_spmm_banded(m, k, n, A.nnz, d.ro, d.ci, d.val, g.dev(b), C)
        spdl.spdl_sddmm_banded(m, k, n, A.nnz, d.ro, d.ci, g.dev(B), g.dev(b), out)
        results.append((C.cpu().numpy(), out.cpu().numpy()))
    assert np.array_equal(results[0][0], results[1][0]) and np.array_equal(results[0][1], results[1][1])
