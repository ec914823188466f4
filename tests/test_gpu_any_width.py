"""Dense widths that are multiples of nothing and operands that start at any element: the kernels that
move 16 bytes per lane take them too, the lane at the end of a row working on the row's last piece.
Sizes at the edges of tiles, slabs and pieces; the arrays lie inside larger ones full of NaN, so that
a value taken from outside shows in the result and a store outside shows in the frame."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need a GPU"
    from tests import gpu_util
    return gpu_util


def framed(a, shift, fill=float("nan")):
    """`a` on the GPU, `shift` elements into a buffer of `fill`; returns (buffer, view, offset)."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    buf = torch.full((t.numel() + 64,), fill, dtype=t.dtype, device="cuda")
    at = 32 + shift
    buf[at:at + t.numel()] = t.view(-1)
    return buf, buf[at:at + t.numel()].view(t.shape), at


def frame_intact(buf, at, count):
    import torch
    edge = torch.cat([buf[:at], buf[at + count:]])
    return bool((edge == 777.0).all())


SPMM_SHAPES = [(4300, 1111, 63, 0.2), (4300, 1111, 66, 0.1), (8192, 300, 127, 0.2), (4100, 777, 129, 0.1),
               (8200, 520, 257, 0.1), (4096, 1030, 1027, 0.1), (4096, 257, 1090, 0.3), (6200, 2048, 33, 0.36)]


@pytest.mark.parametrize("m,k,n,density", SPMM_SHAPES)
@pytest.mark.parametrize("shift", [0, 1])
def test_spmm_slab_kernels_any_width(g, oracle_lib, m, k, n, density, shift):
    import torch
    import paper_2006_10901_amd as spdl
    A = wl.uniform_mask_csr(m, k, density, 7000 + n)
    B = wl.dense(k, n, 7001 + n)
    bias = wl.dense(1, m, 7002 + n)[0]
    C, S = oracle_lib.spmm_bias_relu(m, k, n, A.row_offsets, A.column_indices, A.values, B, bias, False)
    d = g.DevCsr(A)
    _, dB, _ = framed(B, shift)
    cbuf, dC, at = framed(np.full((m, n), np.nan, np.float32), shift, 777.0)
    order = g.dev(spdl.spdl_build_row_order(m, A.row_offsets)) if shift else None
    spdl.spdl_force_variant(0, 2)
    try:
        name = spdl.spdl_variant_name(0, spdl.spdl_select_spmm(m, k, n, A.nnz, 4, dB, dC)["variant"])
        assert name == "slabdma"
        spdl.spdl_spmm_bias_relu(m, k, n, A.nnz, d.ro, d.ci, d.val, order, dB, g.dev(bias), False, dC)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(0, -1)
    g.assert_close(dC.cpu().numpy(), C, S, g.TOL_F32, f"spmm {m}x{k} n={n}")
    assert frame_intact(cbuf, at, m * n)


@pytest.mark.parametrize("n", [33, 63, 127])
@pytest.mark.parametrize("banded", [False, True])
def test_spmm_window_kernel_any_width(g, oracle_lib, n, banded):
    import torch
    import paper_2006_10901_amd as spdl
    A = wl.banded_attention_csr(4099, 256, 0.075, 7050 + n) if banded else wl.uniform_mask_csr(4099, 4300, 0.04, 7050 + n)
    B = wl.dense(A.k, n, 7051 + n)
    C, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    d = g.DevCsr(A)
    _, dB, _ = framed(B, 1)
    cbuf, dC, at = framed(np.full((A.m, n), np.nan, np.float32), 1, 777.0)
    assert spdl.spdl_variant_name(0, spdl.spdl_select_spmm(A.m, A.k, n, A.nnz, 4, dB, dC)["variant"]) == "window"
    spdl.spdl_spmm(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, None, dB, dC)
    torch.cuda.synchronize()
    g.assert_close(dC.cpu().numpy(), C, S, g.TOL_F32, f"window n={n}")
    assert frame_intact(cbuf, at, A.m * n)


@pytest.mark.parametrize("n", [5, 19, 63, 130])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_spmm_row_splitting_with_wide_loads_at_any_width(g, oracle_lib, n, dtype):
    import torch
    import paper_2006_10901_amd as spdl
    m, k = 3000, 2000
    density = 2.2e7 / (m * k * n)
    A = wl.adversarial_csr(m, k, 7100 + n) if density > 0.3 else wl.uniform_mask_csr(m, k, density, 7100 + n)
    A.values = A.values.astype(dtype)
    B = wl.dense(k, n, 7101 + n, dtype)
    C, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    d = g.DevCsr(A)
    _, dB, _ = framed(B, 1)
    cbuf, dC, at = framed(np.full((m, n), np.nan, dtype), 1, 777.0)
    spdl.spdl_force_variant(0, 0)
    try:
        fn = spdl.spdl_spmm_f16 if dtype == np.float16 else spdl.spdl_spmm
        fn(m, k, n, A.nnz, d.ro, d.ci, d.val, None, dB, dC)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(0, -1)
    g.assert_close(dC.cpu().numpy(), C, S, g.TOL_F16 if dtype == np.float16 else g.TOL_F32, f"row splitting n={n}")
    assert frame_intact(cbuf, at, m * n)


@pytest.mark.parametrize("m,n,shift,vec", [(300, 515, 0, 1), (600, 515, 0, 2), (1300, 515, 0, 8), (600, 1030, 0, 8),
                                           (600, 1030, 1, 2), (450, 513, 1, 2), (1500, 1029, 1, 8)])
@pytest.mark.parametrize("lognormal", [False, True])
def test_spmm_row_splitting_in_half_precision_at_odd_elements(g, oracle_lib, m, n, shift, vec, lognormal):
    """Half-precision rows that start at odd elements: 1, 2 or 8 columns per lane by the number of waves, the row's last
    lane on its last columns."""
    import torch
    import paper_2006_10901_amd as spdl
    A = (wl.lognormal_rows_csr if lognormal else wl.uniform_mask_csr)(m, 300, 0.05, 7150 + n)
    A.values = A.values.astype(np.float16)
    B = wl.dense(300, n, 7151 + n, np.float16)
    C, S = oracle_lib.spmm(m, 300, n, A.row_offsets, A.column_indices, A.values, B)
    d = g.DevCsr(A)
    _, dB, _ = framed(B, shift)
    cbuf, dC, at = framed(np.full((m, n), np.nan, np.float16), shift, 777.0)
    spdl.spdl_force_variant(0, 0)
    try:
        assert spdl.spdl_select_spmm(m, 300, n, A.nnz, 2, dB, dC)["vec"] == vec
        spdl.spdl_spmm_f16(m, 300, n, A.nnz, d.ro, d.ci, d.val, None, dB, dC)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(0, -1)
    g.assert_close(dC.cpu().numpy(), C, S, g.TOL_F16, f"row splitting m={m} n={n} shift={shift}")
    assert frame_intact(cbuf, at, m * n)


@pytest.mark.parametrize("n", [1, 8, 16, 20, 64, 100, 128, 200, 256, 300, 515])
@pytest.mark.parametrize("longer", [0, 16, 140])
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
def test_spmm_row_splitting_remainders_of_rows(g, oracle_lib, n, longer, dtype):
    """Rows of every length from empty over whole batches of 8 and 16 to one past them, at the widths where the
    number of columns per lane, of lanes per row and of lane groups sharing a row changes."""
    import torch
    import paper_2006_10901_amd as spdl
    m, k = 517, 400
    lengths = np.arange(m) % 34 + longer
    A = wl.row_lengths_csr(m, k, lengths, 7200 + n)
    A.values = A.values.astype(dtype)
    B = wl.dense(k, n, 7201 + n, dtype)
    C, S = oracle_lib.spmm(m, k, n, A.row_offsets, A.column_indices, A.values, B)
    d = g.DevCsr(A)
    _, dB, _ = framed(B, 0)
    cbuf, dC, at = framed(np.full((m, n), np.nan, dtype), 0, 777.0)
    spdl.spdl_force_variant(0, 0)
    try:
        fn = spdl.spdl_spmm_f16 if dtype == np.float16 else spdl.spdl_spmm
        fn(m, k, n, A.nnz, d.ro, d.ci, d.val, None, dB, dC)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(0, -1)
    g.assert_close(dC.cpu().numpy(), C, S, g.TOL_F16 if dtype == np.float16 else g.TOL_F32, f"row splitting n={n}")
    assert frame_intact(cbuf, at, m * n)


def sddmm_any(g, oracle_lib, A, n, dtype, forced, shift, scaled=False, poke=None):
    import torch
    import paper_2006_10901_amd as spdl
    L, R = wl.dense(A.m, n, 7201 + n, dtype), wl.dense(A.k, n, 7202 + n, dtype)
    if poke:
        poke(L, R)
    with np.errstate(invalid="ignore", over="ignore"):
        ref, S = oracle_lib.sddmm(A.m, A.k, n, A.row_offsets, A.column_indices, L, R)
    d = g.DevCsr(A)
    _, dL, _ = framed(L, shift)
    _, dR, _ = framed(R, shift)
    obuf, out, at = framed(np.full(A.nnz, np.nan, dtype), shift, 777.0)
    spdl.spdl_force_variant(1, forced)
    try:
        chosen = spdl.spdl_variant_name(1, spdl.spdl_select_sddmm(A.m, A.k, n, A.nnz, L.itemsize, dL, dR)["variant"])
        if scaled:
            spdl.spdl_sddmm_scaled(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, dL, dR, out)
        elif dtype == np.float16:
            spdl.spdl_sddmm_f16(A.m, A.k, n, A.nnz, d.ro, d.ci, dL, dR, out)
        else:
            spdl.spdl_sddmm(A.m, A.k, n, A.nnz, d.ro, d.ci, dL, dR, out)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(1, -1)
    assert frame_intact(obuf, at, A.nnz)
    v = A.values.astype(np.float64) if scaled else np.ones(A.nnz)
    return chosen, out.cpu().numpy(), v * ref, np.abs(v) * S


@pytest.mark.parametrize("n", [4, 5, 31, 63, 65, 67, 97, 127, 129, 195, 254, 261, 387, 1001])
@pytest.mark.parametrize("kernel", ["group", "slabdma", "lane", None])
def test_sddmm_any_width(g, oracle_lib, n, kernel):
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(1, v): v for v in range(16) if spdl.spdl_variant_name(1, v)}
    A = wl.uniform_mask_csr(700, 1111, 0.12, 7200 + n)
    for shift, scaled in ((0, False), (1, True)):
        chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float32, -1 if kernel is None else ids[kernel], shift, scaled)
        if kernel and (n <= 128 or n >= 192) and not (kernel == "lane" and 0 < n % 128 < 4):
            assert chosen == kernel
        g.assert_close(got, ref, S, g.TOL_F32, f"sddmm {chosen} n={n} shift={shift}")
    U = wl.adversarial_csr(203, 700, 7203 + n, sorted_cols=False)
    chosen, got, ref, S = sddmm_any(g, oracle_lib, U, n, np.float32, -1 if kernel is None else ids[kernel], 1)
    g.assert_close(got, ref, S, g.TOL_F32, f"sddmm {chosen} n={n}, rows that are not ascending")


@pytest.mark.parametrize("n", [5, 63, 98, 131, 1001])
def test_sddmm_f16_any_width(g, oracle_lib, n):
    A = wl.uniform_mask_csr(300, 500, 0.1, 7300 + n)
    A.values = A.values.astype(np.float16)
    chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float16, -1, 1)
    g.assert_close(got, ref, S, g.TOL_F16, f"sddmm f16 {chosen} n={n}")


@pytest.mark.parametrize("m,k,density", [(300, 500, 0.1), (33, 16, 0.6), (65, 1024, 0.3), (4100, 250, 0.05), (70, 1040, 0.5)])
@pytest.mark.parametrize("n", [8, 9, 15, 34, 255, 257, 263, 519, 1001])
def test_spmm_matrix_core_kernel_any_width(g, oracle_lib, m, k, density, n):
    """One and two tiles per workgroup, panels filled at once and by chunks of 1024 columns, rows that end
    inside a lane's eight columns; empty rows, long rows, rows that are not ascending."""
    import torch
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(0, v): v for v in range(16) if spdl.spdl_variant_name(0, v)}
    for A in (wl.uniform_mask_csr(m, k, density, 7550 + n), wl.adversarial_csr(m, k, 7551 + n, sorted_cols=False),
              wl.adversarial_csr(m, k, 7552 + n)):
        A.values = A.values.astype(np.float16)
        B, bias = wl.dense(k, n, 7553 + n, np.float16), wl.dense(1, m, 7554 + n, np.float16)[0]
        C, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
        ref, S = np.maximum(C.astype(np.float64) + bias.astype(np.float64)[:, None], 0), S + np.abs(bias.astype(np.float64))[:, None]
        d = g.DevCsr(A)
        for shift in (0, 1):
            _, dB, _ = framed(B, shift)
            cbuf, dC, at = framed(np.full((m, n), np.nan, np.float16), shift, 777.0)
            try:
                spdl.spdl_force_variant(0, ids["mfma"])
                assert spdl.spdl_variant_name(0, spdl.spdl_select_spmm(m, k, n, A.nnz, 2, dB, dC)["variant"]) == "mfma"
                spdl.spdl_spmm_bias_relu_f16(m, k, n, A.nnz, d.ro, d.ci, d.val, None, dB, torch.from_numpy(bias).cuda(), 1, dC)
                torch.cuda.synchronize()
            finally:
                spdl.spdl_force_variant(0, -1)
            got = dC.cpu().numpy().astype(np.float64)
            assert np.all(np.abs(got - ref) <= g.TOL_F16 * S + 2e-3 * np.abs(ref) + 1e-6), (m, k, n, shift)
            assert frame_intact(cbuf, at, m * n)


@pytest.mark.parametrize("m,k", [(300, 500), (65, 63), (2600, 320)])
@pytest.mark.parametrize("n", [8, 9, 15, 16, 17, 119, 120, 122, 127, 128, 129, 137, 514, 1001])
def test_sddmm_matrix_core_kernel_any_width(g, oracle_lib, m, k, n):
    """Stages of 16 pieces of 8 columns, of 15 where rows start at odd elements, and the columns left over;
    blocks dealt to the XCDs as regions and (41 x 5 of them) as runs; rows that are not ascending."""
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(1, v): v for v in range(16) if spdl.spdl_variant_name(1, v)}
    for A in (wl.uniform_mask_csr(m, k, 0.15, 7350 + n), wl.adversarial_csr(m, k, 7351 + n, sorted_cols=False)):
        A.values = A.values.astype(np.float16)
        for shift in (0, 1):
            chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float16, ids["mfma"], shift)
            assert chosen == "mfma"
            g.assert_close(got, ref, S, g.TOL_F16, f"sddmm mfma {m}x{k} n={n} shift={shift}")


@pytest.mark.parametrize("n", [63, 127, 261])
@pytest.mark.parametrize("kernel", ["group", "slabdma", "lane"])
def test_sddmm_any_width_keeps_non_finite_values_where_they_belong(g, oracle_lib, n, kernel):
    """An Inf in a column that the last two pieces of a row share, and a NaN in the row after it."""
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(1, v): v for v in range(16) if spdl.spdl_variant_name(1, v)}
    A = wl.uniform_mask_csr(600, 640, 0.1, 7400 + n)

    def poke(L, R):
        L[L == 0] = 1
        R[77, n - 4] = np.inf
        R[78, n - 1] = np.nan
        R[79, 0] = -np.inf
        R[639, n - 2] = np.inf
    chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float32, ids[kernel], 1, poke=poke)
    assert chosen == kernel
    fin = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    assert np.all(np.abs(got[fin] - ref[fin]) <= g.TOL_F32 * S[fin])


def poke_last_pieces(L, R):
    """Infinities and a NaN in columns that the last two pieces of a row share, and in the rows after it."""
    n = R.shape[1]
    L[L == 0] = 1
    R[77, n - 4], R[78, n - 1], R[79, 0], R[639, n - 2] = np.inf, np.nan, -np.inf, np.inf


def assert_same_where_finite(got, ref, tol, atol=0.0):
    fin = np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    assert np.all(np.abs(got[fin] - ref[fin]) <= tol[fin] + atol)


@pytest.mark.parametrize("n", [63, 127, 129, 261])
@pytest.mark.parametrize("kernel", ["group", "mfma"])
def test_sddmm_f16_any_width_keeps_non_finite_values_where_they_belong(g, oracle_lib, n, kernel):
    """Half precision, rows that start two bytes past a multiple of four."""
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(1, v): v for v in range(16) if spdl.spdl_variant_name(1, v)}
    A = wl.uniform_mask_csr(600, 640, 0.1, 7410 + n)
    A.values = A.values.astype(np.float16)
    chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float16, ids[kernel], 1, poke=poke_last_pieces)
    assert chosen == kernel and 0 < np.count_nonzero(~np.isfinite(ref)) < ref.size // 8
    assert_same_where_finite(got.astype(np.float64), ref, g.TOL_F16 * S, g.ATOL_F16_STORE)


@pytest.mark.parametrize("n", [5, 63, 67, 127, 261])
@pytest.mark.parametrize("kernel,dtype", [("rowsplit", np.float32), ("rowsplit", np.float16), ("slabdma", np.float32),
                                          ("window", np.float32)])
def test_spmm_any_width_keeps_non_finite_values_where_they_belong(g, oracle_lib, n, kernel, dtype):
    """Rows of B with infinities and a NaN in the columns that two lanes share reach the rows of A that store them, at
    widths that are multiples of nothing and operands one element off."""
    import torch
    import paper_2006_10901_amd as spdl
    ids = {spdl.spdl_variant_name(0, v): v for v in range(16) if spdl.spdl_variant_name(0, v)}
    A = wl.uniform_mask_csr(600, 640, 0.05, 7420 + n)
    A.values = A.values.astype(dtype)
    A.values[A.values == 0] = 1
    B = wl.dense(640, n, 7421 + n, dtype)
    poke_last_pieces(np.ones((1, n), dtype), B)
    with np.errstate(invalid="ignore", over="ignore"):
        C, S = oracle_lib.spmm(A.m, A.k, n, A.row_offsets, A.column_indices, A.values, B)
    assert 0 < np.count_nonzero(~np.isfinite(C)) < C.size // 4
    d = g.DevCsr(A)
    _, dB, _ = framed(B, 1)
    cbuf, dC, at = framed(np.full((A.m, n), np.nan, dtype), 1, 777.0)
    spdl.spdl_force_variant(0, ids[kernel])
    try:
        chosen = spdl.spdl_select_spmm(A.m, A.k, n, A.nnz, B.itemsize, dB, dC)["variant"]
        assert spdl.spdl_variant_name(0, chosen) == (kernel if kernel != "window" or n <= 128 else "rowsplit")
        fn = spdl.spdl_spmm_f16 if dtype == np.float16 else spdl.spdl_spmm
        fn(A.m, A.k, n, A.nnz, d.ro, d.ci, d.val, None, dB, dC)
        torch.cuda.synchronize()
    finally:
        spdl.spdl_force_variant(0, -1)
    tol = (g.TOL_F16 if dtype == np.float16 else g.TOL_F32) * np.where(np.isfinite(S), S, 0.0)
    assert_same_where_finite(dC.cpu().numpy().astype(np.float64), C, tol, g.ATOL_F16_STORE if dtype == np.float16 else 0.0)
    assert frame_intact(cbuf, at, A.m * n)


@pytest.mark.parametrize("n", [1, 2, 3])
def test_sddmm_of_fewer_than_four_columns_at_any_element(g, oracle_lib, n):
    """An entry per lane: scaled and not, rows that are not ascending, operands one element off, half precision."""
    for A in (wl.uniform_mask_csr(700, 1111, 0.12, 7500 + n), wl.adversarial_csr(203, 700, 7501 + n, sorted_cols=False)):
        for shift, scaled in ((0, False), (1, True)):
            chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float32, -1, shift, scaled)
            assert chosen == "rowstrip"
            g.assert_close(got, ref, S, g.TOL_F32, f"sddmm n={n} shift={shift} scaled={scaled}")
        A.values = A.values.astype(np.float16)
        chosen, got, ref, S = sddmm_any(g, oracle_lib, A, n, np.float16, -1, 1)
        g.assert_close(got, ref, S, g.TOL_F16, f"sddmm f16 n={n}")
