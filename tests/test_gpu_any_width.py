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
