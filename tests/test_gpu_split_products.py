"""fp32 on the bf16 matrix cores (three terms per number): the dense forms of the SDDMM lane and slab kernels, against
the oracle.  Tolerance: a product of terms leaves out less than 2^-23 of it, a sum of n products rounds at most n times:
(n + 8) 2^-24 of the sum of absolute products."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


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


def close(gpu, ref, S, n, what):
    assert np.all(np.isfinite(gpu)), what
    err = np.abs(gpu.astype(np.float64) - ref)
    assert np.all(err <= (n + 8) * 2.0 ** -24 * S + 2.0 ** -149), (what, float(np.max(err / np.maximum(S, 1e-300))))


def mask_csr(m, k, density, seed, odd_rows=True):
    """A uniform mask; with `odd_rows` also empty and full rows, a row with a run of neighbours, rows in no order, duplicates."""
    rng = np.random.default_rng(seed)
    mask = rng.random((m, k)) < density
    if odd_rows:
        mask[[0, m // 2, m - 1]] = False
        mask[[1, m - 2]] = True
        mask[2] = False
        mask[2, k // 3:k // 3 + 200] = True
    ro = np.zeros(m + 1, np.int32)
    ro[1:] = np.cumsum(mask.sum(1))
    ci = np.nonzero(mask)[1].astype(np.int32)
    if odd_rows:
        for i in (5, m // 3, m - 3):
            rng.shuffle(ci[ro[i]:ro[i + 1]])
        ci[ro[7] + 3:ro[7] + 6] = ci[ro[7] + 3]
    values = rng.standard_normal(len(ci)).astype(np.float32)
    return wl.Csr(m, k, ro, ci, values)


def runs_split(A, n):
    import paper_2006_10901_amd as spdl
    spdl.spdl_force_variant(1, 3 if n <= 64 else 5)
    info = spdl.spdl_select_sddmm(A.m, A.k, n, A.nnz, 4, 0, 0)
    return info["lanes_per_row"] == 64 and info["rows_per_block"] == 64


# (rows and columns around whole panels of 64 and whole steps of 256; densities on both sides of one and two sixty-fours
# of look-ahead; widths around whole sixteens, the copies' 32, and the odd five sixteens)
@pytest.mark.parametrize("m,k,density", [(300, 500, 0.8), (321, 513, 0.8), (256, 128, 0.85), (700, 1500, 0.6)])
@pytest.mark.parametrize("n", [4, 7, 16, 17, 31, 32, 33, 64, 65, 75, 80, 81, 96])
def test_sddmm_split_products(g, oracle_lib, force, m, k, density, n):
    A = mask_csr(m, k, density, 9000 + m + n)
    L, R = wl.dense(m, n, 9001 + n), wl.dense(k, n, 9002 + n)
    ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, L, R)
    assert runs_split(A, n)
    close(g.gpu_sddmm(A, L, R, n), ref, S, n, f"{m} x {k}, n = {n}")


@pytest.mark.parametrize("m,k,n,density", [(517, 700, 127, 0.85), (517, 700, 128, 0.85), (4100, 2570, 128, 0.19),
                                           (2049, 2305, 64, 0.12), (1999, 1025, 24, 0.07)])
def test_sddmm_split_products_scaled_and_at_odd_addresses(g, oracle_lib, force, m, k, n, density):
    import torch
    import paper_2006_10901_amd as spdl
    A = mask_csr(m, k, density, 9100 + n)
    L, R = wl.dense(m, n, 9101 + n), wl.dense(k, n, 9102 + n)
    ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, L, R)
    assert runs_split(A, n)
    d = g.DevCsr(A)
    out = torch.full((A.nnz + 2,), float("nan"), device="cuda")
    lpad, rpad = torch.full((m * n + 3,), float("nan"), device="cuda"), torch.full((k * n + 3,), float("nan"), device="cuda")
    lpad[1:1 + m * n], rpad[2:2 + k * n] = g.dev(L).view(-1), g.dev(R).view(-1)
    spdl.spdl_sddmm(m, k, n, A.nnz, d.ro, d.ci, lpad[1:1 + m * n].view(m, n), rpad[2:2 + k * n].view(k, n), out[1:-1])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.isnan(got[0]) and np.isnan(got[-1])
    close(got[1:-1], ref, S, n, f"odd addresses, {m} x {k}, n = {n}")
    spdl.spdl_sddmm_scaled(m, k, n, A.nnz, d.ro, d.ci, d.val, g.dev(L), g.dev(R), out[1:-1])
    torch.cuda.synchronize()
    v = A.values.astype(np.float64)
    close(out[1:-1].cpu().numpy(), v * ref, np.abs(v) * S, n, f"scaled, {m} x {k}, n = {n}")


@pytest.mark.parametrize("n", [24, 75])
def test_sddmm_split_products_keep_non_finite_values_and_the_whole_range(g, oracle_lib, force, n):
    """Infinities and NaN reach the entries that depend on them and no others; numbers that no bf16 term can hold (too large
    for a scaled high term, too small for a low one) cost time, not bits."""
    m, k = 321, 513
    A = mask_csr(m, k, 0.8, 9200 + n)
    L, R = wl.dense(m, n, 9201 + n), wl.dense(k, n, 9202 + n)
    assert runs_split(A, n)
    for scale_l, scale_r in ((2.0 ** -100, 2.0 ** -20), (2.0 ** -126, 1.0), (2.0 ** -126, 2.0 ** 100), (2.0 ** 105, 2.0 ** -90), (2.0 ** 60, 2.0 ** 50)):
        l, r = (L * np.float32(scale_l)).astype(np.float32), (R * np.float32(scale_r)).astype(np.float32)
        ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, l, r)
        # (a denormal product or sum is a multiple of 2^-149)
        got = g.gpu_sddmm(A, l, r, n)
        err = np.abs(got.astype(np.float64) - ref)
        assert np.all(err <= (n + 8) * 2.0 ** -24 * S + n * 2.0 ** -149), (scale_l, scale_r)
    L[3, 1], L[200, n - 1], R[100, 0], R[400, 2], R[512, n - 1] = np.inf, np.nan, -np.inf, np.nan, np.float32(3e38)
    with np.errstate(invalid="ignore", over="ignore"):
        ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, A.column_indices, L, R)
    got = g.gpu_sddmm(A, L, R, n).astype(np.float64)
    inside = np.abs(ref) < 1e38
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and 0 < np.count_nonzero(~inside) < A.nnz // 20
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.all(np.abs(got[inside] - ref[inside]) <= (n + 8) * 2.0 ** -24 * S[inside])


def picked(A, k, parts):
    """Which entries the matrix cores' results are stored for, as the kernel's comments say: the part of an entry's column, if its
    range of the row holds the entry and its cursor comes by; and which entries another part's range holds as well."""
    steps, f32 = -(-k // 256), np.float32
    cols = -(-steps // parts) * 256
    taken, shared = np.zeros(A.nnz, bool), np.zeros(A.nnz, bool)
    for i in range(A.m):
        begin, end = int(A.row_offsets[i]), int(A.row_offsets[i + 1])
        c = A.column_indices[begin:end].astype(np.int64)
        bounds = [0]
        for h in range(1, parts):
            key = h * cols
            at = max(0, min(int(f32(end - begin) * (f32(key) / f32(k))) - 32, end - begin - 64))
            window = c[at:at + 64]
            below = int(np.argmax(window >= key)) if np.any(window >= key) else len(window)
            lo = hi = at + below
            if below == 0 and at > 0:
                lo = 0
            if below == 64:
                hi = end - begin
            while lo < hi:
                mid = (lo + hi) // 2
                lo, hi = (mid + 1, hi) if c[mid] < key else (lo, mid)
            bounds.append(lo)
        bounds.append(end - begin)
        ranges = np.zeros(end - begin, int)
        for h in range(parts):
            ranges[bounds[h]:bounds[h + 1]] += 1
            at = bounds[h]
            for step in range(h * cols // 256, min((h + 1) * cols // 256, steps)):
                while at < bounds[h + 1] and c[at] // 256 == step:
                    taken[begin + at] = True
                    at += 1
        shared[begin:end] = ranges > 1
    return taken, shared


@pytest.mark.parametrize("m,k,n,density", [(320, 2570, 128, 0.8), (320, 1500, 96, 0.8), (515, 4097, 64, 0.5), (300, 5000, 75, 0.6),
                                           (256, 1300, 20, 0.7)])
def test_sddmm_split_products_of_rows_in_no_order_do_not_depend_on_who_stores_last(g, oracle_lib, force, m, k, n, density):
    import paper_2006_10901_amd as spdl
    A = mask_csr(m, k, density, 9300 + n, odd_rows=False)
    L, R = wl.dense(m, n, 9301 + n), wl.dense(k, n, 9302 + n)
    assert runs_split(A, n)
    parts = spdl.spdl_select_sddmm(m, k, n, A.nnz, 4, 0, 0)["grid_y"]
    assert parts > 1
    ascending = g.gpu_sddmm(A, L, R, n)                       # every entry from the matrix cores
    rng = np.random.default_rng(9303)
    order = np.arange(A.nnz)
    for i in range(m):
        row = order[A.row_offsets[i]:A.row_offsets[i + 1]]
        if i % 5 == 1:
            rng.shuffle(row)
        elif i % 5 > 1:                                       # a few ascending runs, exchanged
            runs = np.split(row.copy(), np.sort(rng.integers(0, len(row), int(rng.integers(2, 8)))))
            row[:] = np.concatenate([runs[j] for j in rng.permutation(len(runs))])
    B = wl.Csr(m, k, A.row_offsets, A.column_indices[order].copy(), A.values)
    taken, shared = picked(B, k, parts)
    assert np.count_nonzero(taken & shared) > 200 and not np.all(taken)
    got = g.gpu_sddmm(B, L, R, n)
    ref, S = oracle_lib.sddmm(m, k, n, B.row_offsets, B.column_indices, L, R)
    close(got, ref, S, n, f"{m} x {k}, n = {n}")
    assert np.array_equal(got[taken], ascending[order][taken])
    for _ in range(3):
        assert np.array_equal(g.gpu_sddmm(B, L, R, n), got)


def lane_bounds(c, k, parts, cols):
    """Where the lane kernel's parts begin in a row: sixteen probes around the place that evenly spread columns would give, then
    by sixteenths; rows that are not ascending have some such bounds too."""
    f32, bounds = np.float32, [0]
    for h in range(1, parts):
        key, lo, hi = h * cols, 0, len(c)
        f = f32(key) / f32(k)
        gap = int(f32(0.5) * np.sqrt(max(f32(hi) * f * (f32(1) - f), f32(0)))) + 1
        at = lambda i: min(max(int(f32(len(c)) * f) - ((15 * gap) >> 1) + i * gap, 0), len(c) - 1)
        less = [c[at(i)] < key for i in range(16)] + [False]
        count = less.index(False)
        lo = at(count - 1) + 1 if count > 0 else 0
        hi = max(at(count) if count < 16 else hi, lo)
        while lo < hi:
            step = (hi - lo + 15) >> 4
            count = ([lo + (i + 1) * step - 1 < hi and c[lo + (i + 1) * step - 1] < key for i in range(16)] + [False]).index(False)
            hi = max(min(hi, lo + (count + 1) * step - 1), lo + count * step)
            lo += count * step
        bounds.append(lo)
    return bounds + [len(c)]


@pytest.mark.parametrize("m,k,n,density", [(300, 1500, 100, 0.3), (515, 2570, 200, 0.3), (2500, 1283, 389, 0.1), (300, 1500, 256, 0.5)])
def test_sddmm_lane_kernel_adds_no_chunk_to_what_another_part_has_stored(g, oracle_lib, force, m, k, n, density):
    """Rows of ascending runs, exchanged: the ranges of two parts may overlap, of which one adds the chunks of 128 columns one by
    one and the other stores whole sums."""
    import torch
    import paper_2006_10901_amd as spdl
    A = mask_csr(m, k, density, 9400 + n, odd_rows=False)
    L, R = wl.dense(m, n, 9401 + n), wl.dense(k, n, 9402 + n)
    rng = np.random.default_rng(9403)
    ci = A.column_indices
    for i in range(m):
        row = ci[A.row_offsets[i]:A.row_offsets[i + 1]]
        if i % 5 == 1:
            rng.shuffle(row)
        elif i % 5 > 1:
            runs = np.split(row.copy(), np.sort(rng.integers(0, len(row), int(rng.integers(2, 8)))))
            row[:] = np.concatenate([runs[j] for j in rng.permutation(len(runs))])
    force(1, 5)
    info = spdl.spdl_select_sddmm(m, k, n, A.nnz, 4, 0, 0)
    assert spdl.spdl_variant_name(1, info["variant"]) == "lane" and info["lanes_per_row"] == 2
    parts = info["grid_y"]
    cols = -(-(-(-k // 128)) // parts) * 128
    met = 0
    for i in range(m):
        c = ci[A.row_offsets[i]:A.row_offsets[i + 1]]
        b = lane_bounds(c, k, parts, cols)
        for h in range(parts):
            seg = c[b[h]:b[h + 1]]
            if len(seg) and np.all(np.diff(seg) > 0) and seg[0] >= h * cols and seg[-1] < (h + 1) * cols:
                met += any(o != h and max(b[o], b[h]) < min(b[o + 1], b[h + 1]) for o in range(parts))
    assert met > 0
    ref, S = oracle_lib.sddmm(m, k, n, A.row_offsets, ci, L, R)
    got = g.gpu_sddmm(A, L, R, n)
    close(got, ref, S, n, f"{m} x {k}, n = {n}")
    for _ in range(3):
        assert np.array_equal(g.gpu_sddmm(A, L, R, n), got)
    if n <= 128:
        force(1, -1)
        d, out = g.DevCsr(A), torch.full((A.nnz,), float("nan"), device="cuda")
        spdl.spdl_sddmm_nt(m, k, n, A.nnz, d.ro, d.ci, d.val, g.dev(L), g.dev(np.ascontiguousarray(R.T)), out)
        torch.cuda.synchronize()
        v = A.values.astype(np.float64)
        close(out.cpu().numpy(), v * ref, np.abs(v) * S, n, f"not transposed, {m} x {k}, n = {n}")
