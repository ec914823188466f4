"""Row-splitting SpMM whose rows are shared by lane groups, up to all of a workgroup's, against the oracle.  Tolerance: a chain of at most
as many multiply-adds as the longest row has entries and eight additions of partial sums, (r + 8) 2^-24 of the sum of absolute
products; half precision is rounded once more."""
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
    spdl.spdl_force_variant(0, -1)


def shape(m, k, n, nnz, eb):
    """Lanes of a group, groups per row."""
    import paper_2006_10901_amd as spdl
    s = spdl.spdl_select_spmm(m, k, n, nnz, eb, 0, 0)
    assert spdl.spdl_variant_name(0, s["variant"]) == "rowsplit" and s["block_threads"] == 256
    assert s["grid_x"] == -(-m // s["rows_per_block"]) and s["grid_y"] == -(-n // (s["lanes_per_row"] * s["vec"]))
    return s["lanes_per_row"], 256 // (s["rows_per_block"] * s["lanes_per_row"])


def test_how_many_lane_groups_share_a_row(force):
    force(0, 0)
    assert shape(512, 512, 128, 26214, 4) == (32, 8)                       # 51 entries for 8 groups
    assert shape(512, 512, 128, 512 * 23, 4) == (32, 2) and shape(512, 512, 128, 512 * 15, 4)[1] == 1
    assert shape(1024, 700, 40, 1024 * 48, 4) == (16, 16) and shape(1025, 700, 40, 1025 * 71, 4) == (16, 4)
    assert shape(2048, 700, 40, 2048 * 72, 4) == (16, 16) and shape(2049, 700, 40, 2049 * 300, 4) == (16, 4)
    assert shape(500, 500, 30, 500 * 96, 4) == (8, 32) and shape(500, 500, 30, 500 * 95, 4) == (8, 8)
    assert shape(500, 500, 200, 500 * 100, 4)[1] == 1                      # a group is a wave
    assert shape(500, 900, 200, 500 * 100, 2) == (32, 8)


# (one, two, four and eight groups of a wave and all of a workgroup's; whole and partial last pieces; rows of 0, 1, 2 and all
# columns, in no order, with duplicates; 8 and 32 bounds on a group's batches of eight)
@pytest.mark.gpu
@pytest.mark.parametrize("m,k,density", [(90, 70, 0.4), (515, 300, 0.1), (400, 700, 0.2), (1100, 500, 0.2)])
@pytest.mark.parametrize("n,dtype", [(4, np.float32), (17, np.float32), (31, np.float32), (32, np.float32), (63, np.float32), (64, np.float32), (100, np.float32),
                                     (127, np.float32), (128, np.float32), (130, np.float32), (9, np.float16), (64, np.float16), (127, np.float16), (250, np.float16)])
def test_shared_rows(g, oracle_lib, force, m, k, density, n, dtype):
    import torch
    import paper_2006_10901_amd as spdl
    f16 = dtype == np.float16
    A = odd_csr(m, k, density, 8000 + m)
    A.values = A.values.astype(dtype)
    force(0, 0)
    lanes, groups = shape(m, k, n, A.nnz, 2 if f16 else 4)
    assert groups > 1 or lanes == 64
    B = wl.dense(k, n, 8001 + n, dtype)
    bias = np.random.default_rng(8002).standard_normal(m).astype(dtype)
    d = g.DevCsr(A)
    t = torch.float16 if f16 else torch.float32
    b, c = (torch.full((size + 2,), float("nan"), dtype=t, device="cuda") for size in (k * n, m * n))
    b[1:-1] = g.dev(B).view(-1)
    fn = spdl.spdl_spmm_bias_relu_f16 if f16 else spdl.spdl_spmm_bias_relu
    ref, S = oracle_lib.spmm_bias_relu(m, k, n, A.row_offsets, A.column_indices, A.values.astype(np.float32), B.astype(np.float32), bias.astype(np.float32), True)
    S = S + np.abs(bias.astype(np.float64))[:, None]
    longest = int(np.max(np.diff(A.row_offsets)))
    for order in (None, g.dev(oracle_lib.row_order(m, A.row_offsets))):
        c[1:-1] = float("nan")
        fn(m, k, n, A.nnz, d.ro, d.ci, d.val, order, b[1:-1].view(k, n), g.dev(bias), True, c[1:-1].view(m, n))
        torch.cuda.synchronize()
        got = c.cpu().numpy().astype(np.float64)
        assert np.isnan(got[0]) and np.isnan(got[-1]) and np.all(np.isfinite(got[1:-1]))
        bound = (longest + 8) * 2.0 ** -24 * S + (2.0 ** -11 * np.abs(ref) + 2.0 ** -25 if f16 else 0.0)
        assert np.all(np.abs(got[1:-1].reshape(m, n) - ref) <= bound)
