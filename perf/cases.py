"""Workloads whose speed is followed on one MI355X, each a single call of a public entry point.

The sizes are the five GEMM workloads' (seeded_inputs.CONFIGS), the benchmark's and the tests' own, plus
generic ones at the ends of the ranges: a product with few rows, a mid-sized square one, a small normalisation.
`listed()` names them, `draw()` gives more of the same ranges, `prepare()` makes what a program has in hand
before the call, `run()` is the call, `work()` its minimal traffic and arithmetic, `exact()` the same result
in 64 bits by plain torch.
"""
import math

import torch

import paper_2508_20258_amd as swz

# the largest drawn case of each kind does no more than the largest listed one
MAX_GEMM_FLOPS = 2 * 10000 * 7000 * 4096
MAX_TRANSPOSE_ELEMS = 16384 * 16384      # of two bytes
MAX_ROW_ELEMS = 32768 * 16384
MAX_CHUNKED_ELEMS = 1024 * 65536         # rows cut into chunks: the form for few, long rows


def listed():
    return [
        # products: the smallest workload (latency of one launch), a mid-sized square one that has as many
        # 128-wide tiles as the chip has compute units, the headline size, a projection-shaped one, a ragged one
        dict(name="gemm_512", op="gemm", M=512, N=512, K=512, mode="xcd_groupm"),
        dict(name="gemm_2048", op="gemm", M=2048, N=2048, K=2048, mode="xcd_groupm"),
        dict(name="gemm_4096", op="gemm", M=4096, N=4096, K=4096, mode="xcd_groupm"),
        dict(name="gemm_projection", op="gemm", M=16384, N=2048, K=8192, mode="xcd_groupm"),
        dict(name="gemm_ragged", op="gemm", M=10000, N=7000, K=4096, mode="xcd_groupm"),
        # a product with few rows (a small batch against a large weight matrix): bound by reading B once
        dict(name="gemm_few_rows", op="gemm", M=32, N=8192, K=8192, mode="xcd_groupm"),
        # transposes: the benchmark's size (a power-of-two pitch, beyond the memory-side cache), and four-byte
        # elements at the ragged size of the tests (rows that start in the middle of a line)
        dict(name="transpose_16384", op="transpose", M=16384, N=16384, elem_bytes=2),
        dict(name="transpose32_ragged", op="transpose", M=5800, N=5804, elem_bytes=4),
        # row-wise kernels: the benchmark's largest softmax, its square layer normalisation, its long rows cut into
        # eight chunks, and a normalisation so small that the launch is most of it
        dict(name="softmax_large", op="softmax", M=32768, N=16384, chunks=1, mode="xcd"),
        dict(name="layernorm_8192", op="layernorm", M=8192, N=8192, chunks=1, mode="xcd"),
        dict(name="softmax_long_rows", op="softmax", M=1024, N=65536, chunks=8, mode="xcd"),
        dict(name="layernorm_small", op="layernorm", M=300, N=2048, chunks=1, mode="xcd"),
    ]


def _log_int(rng, lo, hi, multiple=1):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(multiple, v // multiple * multiple)


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm", "gemm", "transpose", "transpose", "softmax", "layernorm", "rows_chunked"])
    if op == "gemm":
        while True:
            M, N, K = _log_int(rng, 1, 16384), _log_int(rng, 64, 16384, 8), _log_int(rng, 64, 16384, 8)
            if 2 * M * N * K <= MAX_GEMM_FLOPS:
                break
        mode = rng.choice(["xcd_groupm", "xcd_groupm", "xcd_groupm", "xcd", "rr"])
        return dict(op="gemm", M=M, N=N, K=K, mode=mode)
    if op == "transpose":
        elem_bytes = rng.choice([2, 2, 4])
        multiple = 16 // elem_bytes
        while True:
            M, N = _log_int(rng, 64, 32768, multiple), _log_int(rng, 64, 32768, multiple)
            if M * N * elem_bytes <= MAX_TRANSPOSE_ELEMS * 2:
                break
        return dict(op="transpose", M=M, N=N, elem_bytes=elem_bytes)
    if op == "rows_chunked":
        op = rng.choice(["softmax", "layernorm"])
        chunks = rng.choice([2, 4, 8, 16])
        while True:
            M, N = _log_int(rng, 1, 4096), _log_int(rng, 4096, 1 << 20, 8)
            if M * N <= MAX_CHUNKED_ELEMS:
                break
        return dict(op=op, M=M, N=N, chunks=chunks, mode="xcd")
    while True:
        M, N = _log_int(rng, 1, 1 << 17), _log_int(rng, 64, 1 << 17, 8)
        if M * N <= MAX_ROW_ELEMS:
            break
    return dict(op=op, M=M, N=N, chunks=1, mode="xcd")


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(m, n, scale):
        x = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
        rows = max(1, (1 << 27) // n)                  # in strips: the 32-bit values of a large matrix need not exist at once
        for i in range(0, m, rows):
            k = min(rows, m - i)
            x[i:i + k] = torch.randn((k, n), device="cuda", generator=g) * scale
        return x

    M, N = case["M"], case["N"]
    if case["op"] == "gemm":                           # activations against a weight matrix of 1/sqrt(K) entries
        return normal(M, case["K"], 1.0), normal(case["K"], N, case["K"] ** -0.5)
    if case["op"] == "transpose":
        if case["elem_bytes"] == 2:
            return (normal(M, N, 1.0),)
        return (torch.randn((M, N), device="cuda", generator=g),)
    if case["op"] == "softmax":                        # logits
        return (normal(M, N, 2.0),)
    return normal(M, N, 2.0), 1.0 + 0.2 * normal(1, N, 1.0)[0], 0.2 * normal(1, N, 1.0)[0]


def prepare(case, seed):
    """Operands, weights and the output buffer, as a program that makes the call again and again keeps them."""
    ins = _inputs(case, seed)
    M, N = case["M"], case["N"]
    shape = (N, M) if case["op"] == "transpose" else (M, N)
    return dict(case=case, ins=ins, out=torch.empty(shape, dtype=ins[0].dtype, device="cuda"))


def run(state):
    case, ins, out = state["case"], state["ins"], state["out"]
    op = case["op"]
    if op == "gemm":
        return swz.gemm(ins[0], ins[1], out, mode=swz.MODES[case["mode"]])
    if op == "transpose":
        return swz.transpose(ins[0], out)
    if op == "softmax":
        return swz.softmax(ins[0], out, chunks=case["chunks"], mode=swz.MODES[case["mode"]])
    return swz.layernorm(ins[0], ins[1], ins[2], out, chunks=case["chunks"], mode=swz.MODES[case["mode"]])


def work(case):
    M, N = case["M"], case["N"]
    if case["op"] == "gemm":
        K = case["K"]
        return {"bytes": 2 * (M * K + K * N + M * N), "flops": 2 * M * N * K}
    if case["op"] == "transpose":
        return {"bytes": 2 * case["elem_bytes"] * M * N, "flops": 0}
    if case["op"] == "softmax":
        return {"bytes": 4 * M * N, "flops": 5 * M * N}
    return {"bytes": 4 * M * N + 4 * N, "flops": 7 * M * N}


def tolerance(case):
    """Products and row-wise results are rounded once to bf16 (half an ulp is 2^-9 to 2^-8 of a value; about 1.7e-3
    in the 2-norm against 64 bits, measured over the listed cases); two correct 32-bit sums of different order round
    some values to neighbouring bf16 numbers, one ulp apart.  A transpose moves bits."""
    if case["op"] == "transpose":
        return "exact"
    return {"rel": 7e-3, "max": 3e-2}


def exact(case, seed):
    ins = _inputs(case, seed)
    op = case["op"]
    if op == "transpose":
        return ins[0].t().contiguous()
    M, N = case["M"], case["N"]
    out = torch.empty((M, N), dtype=torch.float64, device="cuda")
    if op == "gemm":
        torch.matmul(ins[0].double(), ins[1].double(), out=out)
        return out
    rows = max(1, (1 << 26) // N)
    for i in range(0, M, rows):
        x = ins[0][i:i + rows].double()
        if op == "softmax":
            x = torch.exp(x - x.max(dim=1, keepdim=True).values)
            out[i:i + rows] = x / x.sum(dim=1, keepdim=True)
        else:
            d = x - x.mean(dim=1, keepdim=True)
            var = (d * d).mean(dim=1, keepdim=True)
            out[i:i + rows] = d / torch.sqrt(var + 1e-5) * ins[1].double() + ins[2].double()
    return out
