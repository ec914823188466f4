"""fp32 SpMM of dense sparse matrices on the matrix cores (two fp16 terms per number), with numbers of every magnitude: each row of A and each column
of B is taken times a power of two that falls when a larger number comes.  Tolerance: the terms hold a number to 2^-23 of it or 2^-46 of the
largest one of its row or column, of which a product has two; beyond that the bound for four products of terms, as many roundings as the sum has
steps of sixteen columns: (16 (k / 64 + 1) + 16) 2^-24 of the sum of absolute products."""
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
    return B


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "rows and columns", "growing", "falling", "zeros first", "spikes", "tiny", "huge"])
@pytest.mark.parametrize("m,k,n,density", [(4161, 1025, 130, 0.25), (2100, 1300, 331, 0.45)])
def test_split_spmm_of_any_magnitude(g, oracle_lib, kind, m, k, n, density):
    A = odd_csr(m, k, density, 8101 + k)
    B = numbers(kind, A, n)
    assert runs_split(m, k, n, A.nnz)
    ref, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    got = g.gpu_spmm(A, B, n)
    dense = np.zeros((m, k))
    rows = np.repeat(np.arange(m), np.diff(A.row_offsets))
    np.maximum.at(dense, (rows, A.column_indices), np.abs(A.values.astype(np.float64)))
    held = np.zeros((m, k))
    held[rows, A.column_indices] = 1.0
    absB = np.abs(B.astype(np.float64))
    bound = ((16 * (k // 64 + 1) + 16) * 2.0 ** -24 * S + 2.0 ** -149
             + 2.0 ** -45 * (dense.max(1)[:, None] * (held @ absB) + dense.sum(1)[:, None] * absB.max(0)))
    assert np.all(np.isfinite(got)) and np.all(np.abs(got - ref) <= bound)
    assert np.linalg.norm(got - ref) <= 1e-6 * np.linalg.norm(ref)
