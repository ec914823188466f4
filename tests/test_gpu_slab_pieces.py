"""The copy-based slab SpMM kernel's look-ahead, one piece of consecutive pairs per lane, and its rows shared by several lane
groups, against the oracle.  Tolerance: a row of r pairs is a chain of at most r multiply-adds and three additions of partial
sums: (r + 8) 2^-24 of the sum of absolute products."""
import ctypes

import numpy as np
import pytest

import workloads as wl


def choice(m, k, n, nnz):
    import paper_2006_10901_amd as spdl
    s = spdl.spdl_select_spmm(m, k, n, nnz, 4, 0, 0)
    return spdl.spdl_variant_name(0, s["variant"]), s["rows_per_block"], s["block_threads"]


def form(A, n):
    """Of the slab kernel: tiles scanned for one by one, a slab scanned once for several, tiles of 128 columns, panels of 64 rows."""
    import paper_2006_10901_amd as spdl
    return {-1: "shared", 0: "walking", 1: "inner", 2: "wide", 3: "one row"}[ctypes.CDLL(spdl.LIB_PATH).spdl_debug_slab_form(A.m, A.k, n, A.nnz)]


def test_rows_are_shared_where_panels_of_64_leave_the_machine_half_empty():
    assert choice(3004, 2251, 75, int(3004 * 2251 * 0.15)) == ("slabdma", 32, 1024)      # 94 tiles
    assert choice(2048, 8000, 100, int(2048 * 8000 * 0.2)) == ("slabdma", 16, 1024)      # 64 tiles
    assert choice(8192, 10240, 64, int(8192 * 10240 * 0.2)) == ("slabdma", 32, 1024)     # 128 tiles
    assert choice(8320, 10240, 64, int(8320 * 10240 * 0.2)) == ("slabdma", 64, 1024)     # 130 tiles
    # the shapes around the line between the slab kernel and the gathers
    assert choice(2376, 1055, 84, int(2376 * 1055 * 0.107))[0] == "slabdma"
    assert choice(2376, 1055, 84, int(2376 * 1055 * 0.07))[0] != "slabdma"
    assert choice(2048, 4096, 128, 2048 * 400)[0] == "window"
    # a square matrix may be an attention mask
    assert choice(4096, 4096, 64, 1678008)[0] == "window"


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


@pytest.fixture
def force():
    import paper_2006_10901_amd as spdl
    yield spdl.spdl_force_variant
    spdl.spdl_force_variant(0, -1)
    spdl.spdl_force_variant(1, -1)


def odd_csr(m, k, density, seed):
    """A uniform mask with empty and full rows, rows in no order (one of two pairs), duplicates, and a short last row."""
    rng = np.random.default_rng(seed)
    mask = rng.random((m, k)) < density
    mask[[0, m // 2]] = False
    mask[[1, m - 3]] = True
    mask[8] = False
    mask[8, [3, k - 1]] = True
    mask[m - 1] = False
    mask[m - 1, [k - 2, k - 1][: 1 + seed % 2]] = True
    ro = np.zeros(m + 1, np.int32)
    ro[1:] = np.cumsum(mask.sum(1))
    ci = np.nonzero(mask)[1].astype(np.int32)
    for i in (5, m // 3, m - 3):
        rng.shuffle(ci[ro[i]:ro[i + 1]])
    ci[ro[8]:ro[9]] = ci[ro[8]:ro[9]][::-1].copy()
    ci[ro[7] + 3:ro[7] + 6] = ci[ro[7] + 3]
    return wl.Csr(m, k, ro, ci, rng.standard_normal(len(ci)).astype(np.float32))


def run(g, A, n, force, seed, order=None, bias=None):
    """Forced onto the slab kernel, the arrays of A at odd element addresses with nothing but NaN and far columns around."""
    import torch
    import paper_2006_10901_amd as spdl
    B = wl.dense(A.k, n, seed)
    d = g.DevCsr(A)
    ci = torch.full((A.nnz + 2,), 1 << 30, dtype=torch.int32, device="cuda")
    val = torch.full((A.nnz + 2,), float("nan"), device="cuda")
    ci[1:-1], val[1:-1] = d.ci, d.val
    C = torch.full((A.m, n), float("nan"), device="cuda")
    force(0, 2)
    assert choice(A.m, A.k, n, A.nnz)[0] == "slabdma"
    fn = spdl.spdl_spmm if bias is None else spdl.spdl_spmm_bias_relu
    args = (A.m, A.k, n, A.nnz, d.ro, ci[1:-1], val[1:-1], g.dev(order) if order is not None else None, g.dev(B))
    fn(*args, C) if bias is None else fn(*args, g.dev(bias), True, C)
    torch.cuda.synchronize()
    return B, C.cpu().numpy()


def close(A, got, ref, S, what):
    longest = int(np.max(np.diff(A.row_offsets)))
    err = np.abs(got.astype(np.float64) - ref)
    assert np.all(np.isfinite(got)) and np.all(err <= (longest + 8) * 2.0 ** -24 * S), (what, float(np.max(err / np.maximum(S, 1e-300))))


# (tiles of 64 x 64: up to 64, up to 128 and more; eight groups of tiles and more, up to 2048 rows and beyond; densities for one to four pairs per lane; slabs: whole, ragged, fewer than one)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(515, 777, 64), (600, 300, 75), (1030, 515, 260), (2000, 200, 131), (4100, 130, 130), (4100, 513, 260),
                                   (16500, 70, 128), (1100, 260, 700), (2048, 140, 516), (2049, 140, 516)])
@pytest.mark.parametrize("density", [0.02, 0.1, 0.17, 0.3, 0.7])
def test_slab_pieces(g, oracle_lib, force, m, k, n, density):
    A = odd_csr(m, k, density, 7000 + m + int(100 * density))
    order = oracle_lib.row_order(A.m, A.row_offsets)
    B, got = run(g, A, n, force, 7001 + n, order)
    ref, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    close(A, got, ref, S, f"{m} x {k}, n = {n}, {density}")
    _, plain = run(g, A, n, force, 7001 + n)
    assert np.array_equal(plain, got)


def against_the_oracle_with_bias(g, oracle_lib, force, m, k, n, density, forms):
    A = odd_csr(m, k, density, 7200 + m + int(100 * density))
    assert form(A, n) == forms
    bias = np.random.default_rng(7201).standard_normal(m).astype(np.float32)
    B, got = run(g, A, n, force, 7202 + n, oracle_lib.row_order(A.m, A.row_offsets), bias)
    ref, S = oracle_lib.spmm_bias_relu(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B, bias, True)
    close(A, got, ref, S + np.abs(bias)[:, None], f"{m} x {k}, n = {n}, {density}")


# (tiles of 128 columns, two to a workgroup, or five of 64: whole, ragged; one, two and four pairs per lane and
# rows beyond them; rows and columns around whole panels and slabs of 128; the last shape: two pairs of tiles per workgroup)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(4100, 129, 2048), (4096, 260, 2046), (4000, 383, 1985), (2050, 128, 4100), (3970, 90, 2177), (4096, 130, 4092)])
@pytest.mark.parametrize("density", [0.03, 0.1, 0.2])
def test_slab_tiles_of_128_columns(g, oracle_lib, force, m, k, n, density):
    against_the_oracle_with_bias(g, oracle_lib, force, m, k, n, density, "wide" if m in (4000, 4096) else "walking")


# (nine tiles of 128 columns, two to a workgroup and the last one alone; thirteen and nineteen, four to a workgroup and then one, or
# two and one; the last tile of 76, 1, 17 and 35 columns and whole; all of B in one slab, which is then every pair's first and last, and
# in two and three)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(6000, 127, 1100), (6000, 383, 1152), (6582, 128, 1537), (6609, 129, 1544), (4618, 60, 2321), (4641, 129, 2339)])
@pytest.mark.parametrize("density", [0.03, 0.1, 0.2])
def test_slab_odd_numbers_of_tiles_of_128_columns(g, oracle_lib, force, m, k, n, density):
    against_the_oracle_with_bias(g, oracle_lib, force, m, k, n, density, "wide")


# (eight panels of 128 rows, 64 tiles: two tiles of 64 per workgroup, scanned once for both; look-ahead of 32, 48 and 64 pairs, and
# beyond)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(1000, 300, 4096), (1024, 513, 4090), (899, 257, 4095)])
@pytest.mark.parametrize("density", [0.04, 0.1, 0.15, 0.3])
def test_slab_scanned_once_for_two_tiles(g, oracle_lib, force, m, k, n, density):
    A = odd_csr(m, k, density, 7300 + m + int(100 * density))
    assert form(A, n) == ("inner" if density < 0.3 else "walking")
    B, got = run(g, A, n, force, 7302 + n, oracle_lib.row_order(A.m, A.row_offsets))
    ref, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    close(A, got, ref, S, f"{m} x {k}, n = {n}, {density}")


@pytest.mark.gpu
@pytest.mark.parametrize("nnz", [1, 2, 3, 4, 5, 63, 64, 65])
@pytest.mark.parametrize("m,k", [(700, 400), (200, 400), (4200, 60), (66000, 60)])
def test_slab_pieces_of_arrays_shorter_than_a_round(g, oracle_lib, force, m, k, nnz):
    rng = np.random.default_rng(7100 + nnz)
    row = m - 1 if nnz % 2 else m // 2                                # one row has them all
    ro = np.zeros(m + 1, np.int32)
    ro[row + 1:] = nnz
    A = wl.Csr(m, k, ro, np.sort(rng.integers(0, k, nnz)).astype(np.int32), rng.standard_normal(nnz).astype(np.float32))
    bias = rng.standard_normal(m).astype(np.float32)
    for n in (68, 300):
        B, got = run(g, A, n, force, 7101 + n, bias=bias)
        ref, S = oracle_lib.spmm_bias_relu(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B, bias, True)
        close(A, got, ref, S + np.abs(bias)[:, None], f"{m} x {k}, n = {n}, {nnz}")


# (SDDMM: at most 1024 rows and two and a half times as many columns, whose ranges then share an XCD; eight ranges and more, also
# not a multiple of eight; a row order)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,n", [(300, 1100, 132), (1000, 2600, 260), (1024, 2560, 257), (1025, 2700, 132), (130, 3000, 61)])
def test_sddmm_column_ranges_that_share_an_xcd(g, oracle_lib, force, m, k, n):
    import torch
    import paper_2006_10901_amd as spdl
    A = odd_csr(m, k, 0.06, 7400 + m)
    L, R = wl.dense(m, n, 7401 + n), wl.dense(k, n, 7402 + n)
    ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, L, R)
    force(1, 3)
    assert spdl.spdl_variant_name(1, spdl.spdl_select_sddmm(m, k, n, A.nnz, 4, 0, 0)["variant"]) == "slabdma"
    got = g.gpu_sddmm(A, L, R, n)
    err = np.abs(got.astype(np.float64) - ref)
    assert np.all(np.isfinite(got)) and np.all(err <= (n + 8) * 2.0 ** -24 * S + 2.0 ** -149)
    d = g.DevCsr(A)
    out = torch.full((A.nnz,), float("nan"), device="cuda")
    order = oracle_lib.row_order(A.m, A.row_offsets)
    spdl.spdl_sddmm_ordered(m, k, n, A.nnz, d.ro, d.ci, g.dev(order), g.dev(L), g.dev(R), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), got)
