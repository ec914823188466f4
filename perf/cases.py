"""The work a program built on this library has it do, as measurable cases.

A case is one call, or the few calls that belong together, on one sparse layer:

  forward       C = act(A B + bias): SpMM with the row order, with or without the fused epilogue
  input_grad    A^T dC on the cached transposed topology: the values permuted, then SpMM
  weight_grad   the gradient of A's stored values: SDDMM at A's topology
  step          forward and weight_grad of the same layer, one after the other
  attention     one head on a banded mask: SDDMM scores, softmax over rows, SpMM with the values

Shapes are those of the sparse-matrix workloads the repository already carries (workloads.py, the
tests and bench.py): a small layer, weight-sparse recurrent cells, Transformer feed-forward weights,
attention masks and 1x1 convolutions, from a 512 x 512 matrix to 8192 x 10240 and 4096 tokens.
"""
import math

import torch

import paper_2006_10901_amd as spdl

# Each family's range; listed() holds points of it and draw() covers it.
SPARSE_DENSITY = (0.02, 0.30)      # 98 % .. 70 % sparse, the sweep of the recurrent workload


def _case(op, rows, m, k, n, density, dtype="f32", **more):
    c = {"op": op, "rows": rows, "m": m, "k": k, "n": n, "density": density, "dtype": dtype}
    c.update(more)
    return c


def listed():
    return [
        # a small layer: the whole call is a few microseconds, host and launch costs count
        dict(_case("forward", "uniform", 512, 512, 128, 0.10), name="small_forward"),
        dict(_case("weight_grad", "uniform", 512, 512, 128, 0.10), name="small_weight_grad"),
        # weight-sparse recurrent cell, 4 x hidden 2048 by input 8192 + hidden 2048, batch 128: the
        # usual sparsity and the dense end of the sweep
        dict(_case("forward", "uniform", 8192, 10240, 128, 0.10), name="rnn_forward_90"),
        dict(_case("forward", "uniform", 8192, 10240, 128, 0.30), name="rnn_forward_70"),
        dict(_case("weight_grad", "uniform", 8192, 10240, 128, 0.20), name="rnn_weight_grad_80"),
        # a smaller cell with sizes that are multiples of nothing and the last, incomplete batch of an
        # epoch: forward and weight gradient of a training step
        dict(_case("step", "uniform", 3004, 2251, 75, 0.15), name="rnn_ragged_step"),
        # Transformer feed-forward layer, hidden 1024, filter 4096, 4096 tokens: forward with bias and
        # activation, gradient of the input through the transposed weights, gradient of the weights
        dict(_case("forward", "binomial", 4096, 1024, 4096, 0.10, epilogue=True), name="ffn_forward"),
        dict(_case("input_grad", "binomial", 4096, 1024, 4096, 0.10), name="ffn_input_grad"),
        dict(_case("weight_grad", "binomial", 4096, 1024, 4096, 0.10), name="ffn_weight_grad"),
        # one head of sparse attention: sequence 4096, head dimension 64, band of 256 plus scatter
        dict(_case("attention", "banded", 4096, 4096, 64, 0.10, band=256), name="attention_head"),
        # 1x1 convolution in half precision, 64 images of 7 x 7, output channels of unequal length:
        # inference with bias and ReLU, and the weight gradient
        dict(_case("forward", "lognormal", 1024, 1024, 3136, 0.10, dtype="f16", epilogue=True), name="conv_f16_forward"),
        dict(_case("weight_grad", "uniform", 1024, 1024, 3136, 0.10, dtype="f16"), name="conv_f16_weight_grad"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A dense width: mostly padded batches (multiples of 8), a third of them as they come."""
    n = _log(rng, lo, hi)
    return n if rng.random() < 0.34 else max(8, n // 8 * 8)


def draw(rng):
    kind = rng.choice(["small", "rnn", "rnn", "rnn", "ffn", "ffn", "ffn", "attention", "conv", "conv"])
    density = round(math.exp(rng.uniform(math.log(SPARSE_DENSITY[0]), math.log(SPARSE_DENSITY[1]))), 4)
    if kind == "small":
        m, k, n = _log(rng, 256, 1024), _log(rng, 256, 1024), _width(rng, 16, 128)
        return _case(rng.choice(["forward", "weight_grad", "step"]), "uniform", m, k, n, density)
    if kind == "rnn":
        hidden, inputs = _log(rng, 512, 2048), _log(rng, 512, 8192)
        op = rng.choice(["forward", "weight_grad", "step"])
        if op == "step":                                # two calls: half the entries
            density = round(density / 2, 4)
        return _case(op, "uniform", 4 * hidden, inputs + hidden, _width(rng, 32, 128), density)
    if kind == "ffn":
        hidden = _log(rng, 512, 1024)
        m, k = (4 * hidden, hidden) if rng.random() < 0.5 else (hidden, 4 * hidden)
        density = round(rng.uniform(0.05, 0.20), 4)
        n = _width(rng, 256, int(4096 * min(1.0, 0.10 / density)))
        op = rng.choice(["forward", "input_grad", "weight_grad"])
        return _case(op, "binomial", m, k, n, density, epilogue=op == "forward")
    if kind == "attention":
        seq = _log(rng, 1024, 4096)
        density = round(rng.uniform(0.08, 0.12) * max(1.0, 2048 / seq) + 256.0 / seq * 0.5, 4)
        return _case("attention", "banded", seq, seq, rng.choice([32, 64, 64, 96, 128]), density, band=256)
    m, k = _log(rng, 256, 1024), _log(rng, 256, 1024)
    n = rng.randint(1, 64) * rng.choice([49, 49, 49, 48, 56])
    op = rng.choice(["forward", "weight_grad"])
    return _case(op, rng.choice(["uniform", "lognormal"]), m, k, n, density, dtype="f16", epilogue=op == "forward")


def _entries(case):
    return int(case["density"] * case["m"] * case["k"])


def _topology(case, gen):
    """CSR topology of the case's mask: offsets and ascending column indices, on the GPU.  Every mask
    of a case has the same number of entries: drawn with a slightly larger probability, then thinned."""
    m, k = case["m"], case["k"]
    always, free = torch.zeros((), dtype=torch.bool, device="cuda"), _entries(case)
    p = torch.full((), free / (m * k), device="cuda")
    if case["rows"] == "lognormal":                     # row lengths of coefficient of variation about 1.3
        p = torch.exp(torch.randn((m, 1), generator=gen, device="cuda"))
    elif case["rows"] == "banded":
        i, j = torch.arange(m, device="cuda")[:, None], torch.arange(k, device="cuda")[None, :]
        dist = (i - j).abs()
        always = dist <= case["band"] // 2
        free -= int(always.sum())
        p = torch.where(always, 0.0, 1.0 / dist.clamp(min=1).float())
    p = p.expand(m, k if p.dim() and p.shape[-1] == k else 1)
    for _ in range(8):                                  # scale to the wanted mean, probabilities at most 1
        p = (p * (free / (float(p.mean()) * m * k))).clamp(max=1.0)
    u = torch.rand((m, k), generator=gen, device="cuda")
    more = 1.0 + 8.0 / math.sqrt(free + 1.0)
    while True:
        drawn = torch.nonzero(((u < p * more) & ~always).view(-1))[:, 0]
        if drawn.numel() >= free:
            break
        more *= 1.02
    keep = torch.zeros((m, k), dtype=torch.bool, device="cuda") | always
    keep.view(-1)[drawn[torch.randperm(drawn.numel(), generator=gen, device="cuda")[:free]]] = True
    ro = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    ro[1:] = torch.cumsum(keep.sum(dim=1, dtype=torch.int32), 0)
    return ro, torch.nonzero(keep)[:, 1].to(torch.int32).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    m, k, n, op = case["m"], case["k"], case["n"], case["op"]
    dt = torch.float16 if case["dtype"] == "f16" else torch.float32
    ro, ci = _topology(case, gen)
    nnz = int(ci.numel())

    def normal(*shape, sigma=1.0):
        return (torch.randn(shape, generator=gen, device="cuda") * sigma).to(dt)

    s = {"op": op, "f16": dt == torch.float16, "dims": (m, k, n, nnz), "ro": ro, "ci": ci}
    ro_host = ro.cpu().numpy()
    if op == "attention":
        s.update(Q=normal(m, n), K=normal(k, n), V=normal(k, n), scale=1.0 / math.sqrt(n),
                 probs=torch.empty(nnz, device="cuda"), C=torch.empty((m, n), device="cuda"))
        return s
    s["values"] = normal(nnz, sigma=1.0 if s["f16"] else 0.02)
    s["order"] = torch.from_numpy(spdl.spdl_build_row_order(m, ro_host)).cuda()
    if op in ("forward", "step"):
        s.update(B=normal(k, n), C=torch.empty((m, n), dtype=dt, device="cuda"))
        s["bias"] = normal(m) if case.get("epilogue") else None
    if op in ("weight_grad", "step"):
        s.update(L=normal(m, n), R=s["B"] if op == "step" else normal(k, n),
                 grad=torch.empty(nnz, dtype=dt, device="cuda"))
    if op == "input_grad":
        t_ro, t_ci, perm = spdl.spdl_build_transpose_host(m, k, nnz, ro_host, ci.cpu().numpy())
        s.update(t_ro=torch.from_numpy(t_ro).cuda(), t_ci=torch.from_numpy(t_ci).cuda(),
                 perm=torch.from_numpy(perm).cuda(), t_values=torch.empty_like(s["values"]),
                 t_order=torch.from_numpy(spdl.spdl_build_row_order(k, t_ro)).cuda(),
                 dC=normal(m, n), dB=torch.empty((k, n), dtype=dt, device="cuda"))
    return s


def run(s):
    m, k, n, nnz = s["dims"]
    op = s["op"]
    if op == "attention":
        spdl.spdl_sddmm_banded(m, k, n, nnz, s["ro"], s["ci"], s["Q"], s["K"], s["probs"])
        spdl.spdl_csr_softmax(m, nnz, s["ro"], s["probs"], s["scale"], s["probs"])
        spdl.spdl_spmm_banded(m, k, n, nnz, s["ro"], s["ci"], s["probs"], s["V"], s["C"])
        return {"probabilities": s["probs"], "context": s["C"]}
    if op == "input_grad":
        spdl.spdl_permute_values(nnz, 4, s["perm"], s["values"], s["t_values"])
        spdl.spdl_spmm(k, m, n, nnz, s["t_ro"], s["t_ci"], s["t_values"], s["t_order"], s["dC"], s["dB"])
        return {"t_values": s["t_values"], "dB": s["dB"]}
    out = {}
    if op in ("forward", "step"):
        if s["bias"] is not None:
            f = spdl.spdl_spmm_bias_relu_f16 if s["f16"] else spdl.spdl_spmm_bias_relu
            f(m, k, n, nnz, s["ro"], s["ci"], s["values"], s["order"], s["B"], s["bias"], True, s["C"])
        else:
            f = spdl.spdl_spmm_f16 if s["f16"] else spdl.spdl_spmm
            f(m, k, n, nnz, s["ro"], s["ci"], s["values"], s["order"], s["B"], s["C"])
        out["C"] = s["C"]
    if op in ("weight_grad", "step"):
        f = spdl.spdl_sddmm_f16 if s["f16"] else spdl.spdl_sddmm
        f(m, k, n, nnz, s["ro"], s["ci"], s["L"], s["R"], s["grad"])
        out["grad"] = s["grad"]
    return out


def work(case):
    m, k, n, op = case["m"], case["k"], case["n"], case["op"]
    eb = 2 if case["dtype"] == "f16" else 4
    nnz = _entries(case)
    topology = 4 * nnz + 4 * (m + 1)
    dense = eb * n * (m + k)
    # each input read once, each output written once; SpMM also reads the row order
    spmm = {"bytes": topology + eb * nnz + 4 * m + dense + (eb * m if case.get("epilogue") else 0), "flops": 2 * nnz * n}
    sddmm = {"bytes": topology + eb * nnz + dense, "flops": 2 * nnz * n}
    parts = {"forward": [spmm], "weight_grad": [sddmm],
             # B and the topology serve both
             "step": [spmm, {"bytes": sddmm["bytes"] - topology - eb * n * k, "flops": sddmm["flops"]}],
             # the permutation reads the values once more and writes them
             "input_grad": [spmm, {"bytes": 12 * nnz, "flops": 0}],
             # scores and probabilities pass from call to call through memory
             "attention": [sddmm, {"bytes": 8 * nnz, "flops": 5 * nnz}, spmm]}[op]
    return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}


def tolerance(case):
    # fp32 sums of up to a few thousand products; binary16 results are rounded once from fp32 sums
    return {"rel": 1e-3} if case["dtype"] == "f16" else {"rel": 1e-5}
