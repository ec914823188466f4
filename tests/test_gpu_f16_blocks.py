"""Mixed-precision SDDMM on the matrix cores, blocks of every size, against the oracle.  Tolerance: n products and sums in fp32, (n + 8) 2^-24 of the sum
of absolute products, and the rounding to half precision, 2^-11 of the result or 2^-25."""
import numpy as np
import pytest

import workloads as wl
from tests.test_gpu_split_products import mask_csr

pytestmark = pytest.mark.gpu


@pytest.fixture
def g():
    from tests import gpu_util
    return gpu_util


@pytest.fixture(autouse=True)
def force():
    import paper_2006_10901_amd as spdl
    spdl.spdl_force_variant(1, 4)
    yield
    spdl.spdl_force_variant(1, -1)


# (rows and columns around whole blocks, and on both sides of where a size's blocks are as many as compute units; widths around pieces of 8, tails,
# stages of 128 and 256 and of those less the overlapping piece, one stage more and fewer than the ring holds)
@pytest.mark.parametrize("m,k,cols", [(230, 300, 32), (512, 512, 32), (513, 257, 32), (511, 993, 32), (1025, 385, 32), (897, 610, 64), (1024, 577, 64)])
@pytest.mark.parametrize("n", [8, 9, 16, 23, 120, 135, 247, 248, 256, 257, 264, 505, 768, 777, 1025, 1288])
def test_f16_blocks(g, oracle_lib, m, k, cols, n):
    import torch
    import paper_2006_10901_amd as spdl
    A = mask_csr(m, k, 0.06, 9800 + m + n)
    L, R = (wl.dense(m, n, 9801 + n) / 4).astype(np.float16), (wl.dense(k, n, 9802 + n) / 4).astype(np.float16)
    info = spdl.spdl_select_sddmm(m, k, n, A.nnz, 2, 0, 0)
    assert info["grid_y"] == -(-k // cols) and info["rows_per_block"] == (32 if max(m, k) <= 513 else 64)
    ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, L, R)
    d = g.DevCsr(A)
    # operands at odd element addresses and at even ones, nothing but NaN around
    for at in (1, 4):
        lpad = torch.full((m * n + 8,), float("nan"), device="cuda", dtype=torch.float16)
        rpad = torch.full((k * n + 8,), float("nan"), device="cuda", dtype=torch.float16)
        lpad[at:at + m * n], rpad[4:4 + k * n] = g.dev(L).view(-1), g.dev(R).view(-1)
        out = torch.full((A.nnz + 2,), float("nan"), device="cuda", dtype=torch.float16)
        spdl.spdl_sddmm_f16(m, k, n, A.nnz, d.ro, d.ci, lpad[at:at + m * n].view(m, n), rpad[4:4 + k * n].view(k, n), out[1:-1])
        torch.cuda.synchronize()
        got = out.cpu().numpy().astype(np.float64)
        assert np.isnan(got[0]) and np.isnan(got[-1])
        assert np.all(np.abs(got[1:-1] - ref) <= (n + 8) * 2.0 ** -24 * S + 2.0 ** -11 * np.abs(ref) + 2.0 ** -25)
