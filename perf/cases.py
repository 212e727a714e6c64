"""The reduction-to-all calls that the performance work measures.

A case is one `dpar_allreduce` call (or, with `entry`, one of the other public
entry points) on p ranks of m elements: int32 SUM and MAX, fp32 SUM and the
2x2 uint32 matrix product; separate outputs or in place; rows on cache-line
boundaries or packed; the block count of the sqrt(m log2 p) rule (b = 0) or
the paper's fixed blocks of 16000 elements.
"""

import torch

from paper_2109_12626_amd import dpar

_ELEM = {"int32": 4, "float32": 4, "u32mat2x2": 16}
# value ranges of the repository's workloads
_INT_LO, _INT_HI = -(1 << 20), 1 << 20


def _case(name, p, m, dtype, op, b=0, alg="dual", exec="auto", entry="call",
          pitch=1, in_place=False):
    """entry: "call" (dpar_allreduce on kept pointer arrays), "noalloc" (its
    allocation-free variant), "tensor" (the tensor front end, which marshals
    the rows on every call).  pitch: rows start at multiples of this many
    elements (1: packed; 128: as p separate allocations would)."""
    c = {"p": p, "m": m, "dtype": dtype, "op": op, "b": b, "alg": alg,
         "exec": exec, "entry": entry, "pitch": pitch, "in_place": in_place}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a few ranks' scalars and short vectors (counters,
        # loss terms, small layers) reduced inside a step; launch latency
        _case("p7_m1000", 7, 1000, "int32", "sum", b=4),
        # the paper's Table 2, a short count: 288 processes, 3.5 KB each
        _case("p288_m875", 288, 875, "int32", "sum", b=1, pitch=128),
        # all processes of the paper's machine, short vectors, in place (the
        # paper's single array Y)
        _case("p1152_m1024_max_inplace", 1152, 1024, "int32", "max",
              in_place=True),
        # many ranks with 16 KB each: the latency-bound to bandwidth-bound
        # crossover at the most ranks
        _case("p4608_m4096", 4608, 4096, "int32", "sum"),
        # ragged: packed rows whose length is odd, so every row starts at
        # another alignment
        _case("p300_m100003_f32", 300, 100003, "float32", "sum"),
        # one rank per node of the paper's machine, 4 MB each, through the
        # tensor front end
        _case("p36_m2^20", 36, 1 << 20, "int32", "sum", entry="tensor"),
        # the non-commutative operator
        _case("p64_m2^18_matmul", 64, 1 << 18, "u32mat2x2", "matmul", b=32),
        # all processes of the paper's machine, 256 KB each
        _case("p1152_m2^16", 1152, 1 << 16, "int32", "sum"),
        # the paper's Table 2 count of 250000 ints with the algorithm's whole
        # round structure, down-phase included
        _case("p288_m250000_rounds", 288, 250000, "int32", "sum", b=16,
              exec="rounds", pitch=128),
        # eight ranks with 64 MB each: gradients of a data-parallel step
        _case("p8_m2^24_f32", 8, 1 << 24, "float32", "sum"),
        # the paper's Table 2, a long count (8.5 MB per process) in its blocks
        # of 16000 elements
        _case("p288_m2125000", 288, 2125000, "int32", "sum", b=133,
              pitch=128),
        # the headline: all processes of the paper's machine, 16 MB each
        _case("p1152_m2^22_f32", 1152, 1 << 22, "float32", "sum"),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    dtype, op = rng.choice([("int32", "sum"), ("int32", "max"),
                            ("float32", "sum"), ("float32", "sum"),
                            ("u32mat2x2", "matmul")])
    exec = "rounds" if rng.random() < 0.1 else "auto"
    # whole calls from 28 KB to 16 GB read; the round-structured executor,
    # which launches a kernel for every block, from 36 ranks on up to 0.5 GB
    if exec == "rounds":
        p = int(round(_log_uniform(rng, 36, 1152)))
        total = _log_uniform(rng, 28e3, 0.5e9)
    else:
        p = int(round(_log_uniform(rng, 2, 4608)))
        total = _log_uniform(rng, 28e3, 16e9)
    m = max(1, min(int(total / (p * _ELEM[dtype])), 1 << 28))
    if rng.random() < 0.5:
        m = max(1, m // 64 * 64)   # whole cache lines; else as it falls
    b = -(-m // 16000) if exec == "rounds" else \
        rng.choice([0, 0, 1, -(-m // 16000)])
    alg = "dual" if rng.random() < 0.7 else \
        rng.choice(["single", "reduce_bcast"])
    entry = "call"
    if exec == "auto" and alg == "dual":
        entry = rng.choice(["call", "call", "tensor", "noalloc"])
    return _case(None, p, m, dtype, op, b=b, alg=alg, exec=exec, entry=entry,
                 pitch=rng.choice([1, 128]),
                 in_place=op != "sum" and rng.random() < 0.5)


def _inputs(case, seed):
    """[p, ld] values on the GPU; a rank's vector is the first m of a row
    (4 words per matrix)."""
    p, m, pitch = case["p"], case["m"], case["pitch"]
    words = _ELEM[case["dtype"]] // 4
    ld = -(-m // pitch) * pitch * words
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["dtype"] == "float32":
        return torch.randn((p, ld), generator=g, device="cuda")
    lo, hi = (_INT_LO, _INT_HI + 1) if words == 1 else (-(1 << 31), 1 << 31)
    return torch.randint(lo, hi, (p, ld), generator=g, device="cuda",
                         dtype=torch.int32)


def prepare(case, seed):
    m = case["m"] * (_ELEM[case["dtype"]] // 4)
    x = _inputs(case, seed)
    y = x if case["in_place"] else torch.empty_like(x)
    state = dict(case, x=x[:, :m], y=y[:, :m],
                 stream=torch.cuda.current_stream())
    if case["entry"] != "tensor":
        state["xs"], state["ys"] = dpar.rows(x), dpar.rows(y)
    return state


def run(s):
    """One reduction-to-all; returns the p output vectors ([p, m], or
    [p, 4 m] words for matrices)."""
    if s["entry"] == "tensor":
        return dpar.allreduce(s["x"], s["y"], s["dtype"], s["op"], s["b"],
                              stream=s["stream"])
    if s["entry"] == "noalloc":
        dpar.dpar_allreduce_noalloc(s["xs"], s["ys"], s["p"], s["m"],
                                    s["dtype"], s["op"], s["b"], s["stream"])
    elif s["exec"] == "auto" and s["alg"] == "dual":
        dpar.dpar_allreduce(s["xs"], s["ys"], s["p"], s["m"], s["dtype"],
                            s["op"], s["b"], s["stream"])
    else:
        dpar.dpar_allreduce_opt(s["xs"], s["ys"], s["p"], s["m"], s["dtype"],
                                s["op"], s["b"], s["alg"], s["exec"],
                                stream=s["stream"])
    return s["y"]


def work(case):
    """Every input read once, every output written once; one operator
    application per element and rank (12 integer operations per matrix)."""
    n = case["p"] * case["m"]
    return {"bytes": 2 * n * _ELEM[case["dtype"]],
            "flops": n * (12 if case["op"] == "matmul" else 1)}


def tolerance(case):
    """The association of every operator application is part of the
    interface, so fp32 results are the same bit for bit as well."""
    return "exact"


def exact(case, seed):
    x = _inputs(case, seed)
    p, m = case["p"], case["m"]
    if case["op"] == "matmul":
        a = x.view(p, -1, 4)[:, :m]
        y = a[0].to(torch.int64) & 0xFFFFFFFF
        for i in range(1, p):   # 64-bit products wrap mod 2^64, then mod 2^32
            r = a[i].to(torch.int64) & 0xFFFFFFFF
            y = torch.stack((y[:, 0] * r[:, 0] + y[:, 1] * r[:, 2],
                             y[:, 0] * r[:, 1] + y[:, 1] * r[:, 3],
                             y[:, 2] * r[:, 0] + y[:, 3] * r[:, 2],
                             y[:, 2] * r[:, 1] + y[:, 3] * r[:, 3]),
                            1) & 0xFFFFFFFF
        y = y.to(torch.int32).reshape(-1)   # low 32 bits
    else:
        x = x[:, :m]
        wide = torch.float64 if case["dtype"] == "float32" else torch.int64
        y = x[0].to(wide)
        for i in range(1, p):
            r = x[i].to(wide)
            y = torch.maximum(y, r) if case["op"] == "max" else y + r
        if wide == torch.int64:
            y = y.to(torch.int32)           # wraps mod 2^32
    return y.expand(p, -1)
