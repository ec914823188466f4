"""SDDMM of few entries in the nonzero-split kernel, strips of four entries, against the oracle.  Tolerance: a chain of at most n
multiply-adds and four additions of partial sums, (n + 8) 2^-24 of the sum of absolute products; half precision is rounded once more."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_slab_pieces import odd_csr


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


@pytest.fixture
def force():
    import paper_2006_10901_amd as spdl
    yield spdl.spdl_force_variant
    spdl.spdl_force_variant(1, -1)


def strips(m, k, n, nnz, eb):
    """Entries per wave, waves per workgroup, workgroups."""
    import paper_2006_10901_amd as spdl
    s = spdl.spdl_select_sddmm(m, k, n, nnz, eb, 0, 0)
    assert spdl.spdl_variant_name(1, s["variant"]) in ("group", "rowstrip") and s["lanes_per_row"] == 16      # (rowstrip: fp32 widths of 129 .. 191 that are no multiple of four)
    return s["rows_per_block"], s["block_threads"] // 64, s["grid_x"]


def test_few_entries_take_strips_of_four(force):
    assert strips(512, 512, 128, 26214, 4) == (16, 1, 1639)
    force(1, 1)
    for n, sixteen, thirty_two in ((64, 50000, 400000), (128, 100000, 400000), (256, 80000, 400000)):
        assert strips(20000, 300, n, sixteen, 4) == (16, 1, sixteen // 16) and strips(20000, 300, n, sixteen + 1, 4)[:2] == (32, 1)
        assert strips(20000, 300, n, thirty_two, 4)[:2] == (32, 1) and strips(20000, 300, n, thirty_two + 1, 4)[:2] == (64, 4)
    assert strips(500, 300, 64, 60000, 4)[:2] == (64, 4) and strips(500, 300, 100, 120000, 4)[:2] == (32, 1)     # long rows
    assert strips(500, 300, 64, 5000, 2)[:2] == (64, 4) and strips(500, 300, 65, 5000, 2)[:2] == (16, 1)


def against_the_oracle(g, oracle_lib, A, n, dtype, scaled):
    import torch
    import paper_2006_10901_amd as spdl
    f16 = dtype == np.float16
    A.values = A.values.astype(dtype)
    L, R = wl.dense(A.m, n, 7801 + n, dtype), wl.dense(A.k, n, 7802 + n, dtype)
    ref, S = oracle_lib.sddmm(A.m, A.k, n, A.row_offsets, A.column_indices, L, R)
    d = g.DevCsr(A)
    t = torch.float16 if f16 else torch.float32
    out, l, r = (torch.full((size + 2,), float("nan"), dtype=t, device="cuda") for size in (A.nnz, A.m * n, A.k * n))
    l[1:-1], r[1:-1] = g.dev(L).view(-1), g.dev(R).view(-1)
    args = (l[1:-1].view(A.m, n), r[1:-1].view(A.k, n), out[1:-1])
    if scaled:
        fn = spdl.spdl_sddmm_scaled_f16 if f16 else spdl.spdl_sddmm_scaled
        fn(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, *args)
        v = A.values.astype(np.float64)
        ref, S = v * ref, np.abs(v) * S
    else:
        fn = spdl.spdl_sddmm_f16 if f16 else spdl.spdl_sddmm
        fn(A.m, A.k, n, A.nnz, d.ro, d.ci, *args)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert np.isnan(got[0]) and np.isnan(got[-1]) and np.all(np.isfinite(got[1:-1]))
    bound = (n + 8) * 2.0 ** -24 * S + (2.0 ** -11 * np.abs(ref) + 2.0 ** -25 if f16 else 2.0 ** -149)
    assert np.all(np.abs(got[1:-1] - ref) <= bound)


# (columns around whole pieces of four, sixty-fours and pairs of those; entries for 16 and 32 per wave, the latter in long rows (65 .. 128 columns; the
# other widths take strips of sixteen there) and in short ones; empty and full rows, rows in no order and duplicates; every array at odd elements)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,density", [(90, 70, 0.1), (515, 300, 0.1), (400, 700, 0.4), (4000, 300, 0.08)])
@pytest.mark.parametrize("n,dtype", [(4, np.float32), (7, np.float32), (63, np.float32), (64, np.float32), (65, np.float32), (127, np.float32),
                                     (128, np.float32), (129, np.float32), (260, np.float32), (67, np.float16), (128, np.float16), (189, np.float16)])
def test_strips_of_four(g, oracle_lib, force, m, k, density, n, dtype):
    A = odd_csr(m, k, density, 7800 + m)
    force(1, 1)
    both = 64 < n <= 128
    want = ((32, 1) if both else (64, 4)) if m == 400 else ((16, 1) if both else (32, 1)) if m == 4000 else (16, 1)
    assert strips(m, k, n, A.nnz, np.dtype(dtype).itemsize)[:2] == want
    against_the_oracle(g, oracle_lib, A, n, dtype, scaled=n % 2 == 0)


@pytest.mark.gpu
@pytest.mark.parametrize("nnz", [1, 3, 4, 5, 15, 16, 17, 63, 65])
def test_strips_of_four_with_hardly_any_entries(g, oracle_lib, force, nnz):
    rng = np.random.default_rng(7900 + nnz)
    m, k = 300, 40
    for rows in (rng.integers(0, m, nnz), np.full(nnz, m - 1), np.arange(nnz) * 4 % m):
        ro = np.zeros(m + 1, np.int32)
        ro[1:] = np.cumsum(np.bincount(rows, minlength=m))
        A = wl.Csr(m, k, ro, rng.integers(0, k, nnz).astype(np.int32), rng.standard_normal(nnz).astype(np.float32))
        force(1, 1)
        for n in (20, 100):
            against_the_oracle(g, oracle_lib, A, n, np.float32, scaled=False)
