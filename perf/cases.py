"""Performance cases of the per-rank tensor-parallel GEMMs: one pass is one call of a public entry point.

The shapes are one rank's share of an MLP under tensor parallelism, as in the stated configurations of
`paper_2511_13940_amd/workloads.py` (cfg1 .. cfg5), from a decode step of a few dozen tokens over prefill chunks of one or
two thousand to the full 8192- and 16384-token passes.  Peers' data (chunks of A, partial slots, reduced rows) is in place
with its flags set, as in `bench.py`'s timed step.  All dimensions are global (M tokens, N columns, K reduction length of the
unsharded GEMM).

Case fields: op (entry point without `pk_`), P, rank, M, N, K, dtype ("bf16" / "fp8"), layout of the second operand ("kn" /
"nk"), act (all-gather ops), slots (element type of the partial slots), overlap (the reduce beside the GEMM).
"""
import math

import torch

from paper_2511_13940_amd import pk

READY = 0x7FFFFFFF            # a flag that is ready for every epoch: the peers' data has landed


def _case(name, op, P, rank, M, N, K, dtype="bf16", layout="kn", act="none", slots="f32", overlap=False):
    c = {"op": op, "P": P, "rank": rank, "M": M, "N": N, "K": K, "dtype": dtype, "layout": layout, "act": act, "slots": slots,
         "overlap": overlap}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the smallest call (cfg1): launches and latency are all of it
        _case("rs_256", "gemm_rs", 2, 0, 256, 256, 512),
        # one decode step of 64 sequences through a 70B-class MLP under 8-way tensor parallelism: up-projection ...
        _case("ag_decode_64", "ag_gemm", 8, 0, 64, 28672, 8192, act="silu"),
        # ... and down-projection with the all-reduce that a decode step ends with
        _case("ar_decode_64", "gemm_ar", 8, 3, 64, 8192, 28672),
        # a middle-sized layer (cfg2)
        _case("ag_2048", "ag_gemm", 4, 1, 2048, 4096, 2048),
        # a prefill chunk of 1024 tokens through the down-projection of the 70B-class MLP
        _case("rs_chunk_1024", "gemm_rs", 8, 2, 1024, 8192, 28672),
        # a batch of ragged length, widths that are no tile multiple, the weight stored as a linear layer keeps it
        _case("ag_ragged_1512", "ag_gemm", 8, 5, 1512, 13760, 5120, layout="nk", act="gelu_tanh"),
        # 8-bit operands, a prefill chunk of 2048 tokens through the up-projection
        _case("ag_fp8_2048", "ag_gemm", 8, 7, 2048, 28672, 8192, dtype="fp8"),
        # the scatter and the gather along the last dimension, activations sharded by columns; ragged rows, bf16 slots
        _case("rs_cols_1000", "gemm_rs_cols", 4, 1, 1000, 8192, 11008, slots="bf16"),
        _case("ag_k_4096", "ag_gemm_k", 8, 4, 4096, 14336, 4096),
        # the full passes over 8192 tokens of the 70B-class MLP (cfg4, cfg3): what the benchmark's step runs
        _case("ag_8192", "ag_gemm", 8, 0, 8192, 28672, 8192),
        _case("rs_8192", "gemm_rs", 8, 0, 8192, 8192, 28672, overlap=True),
        # the largest call, 8-bit operands (cfg5)
        _case("rs_fp8_16384", "gemm_rs", 8, 0, 16384, 16384, 16384, dtype="fp8", overlap=True),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(x, of):
    return max(1, round(x / of)) * of


def _cost(c):
    """Rough microseconds, to keep drawn cases under the largest listed one."""
    w = work(c)
    return w["flops"] / (2.0e9 if c["dtype"] == "fp8" else 1.0e9) + w["bytes"] / 5.0e6


def draw(rng):
    """One more call: tokens 16 .. 16384, hidden size 256 .. 16384, one rank's inner width 256 .. 8192."""
    most = max(_cost(c) for c in listed())
    while True:
        op = rng.choice(["gemm_rs", "gemm_rs", "ag_gemm", "ag_gemm", "gemm_ar", "gemm_rs_cols", "ag_gemm_k"])
        dtype = rng.choice(["bf16", "bf16", "fp8"])
        P = rng.choice([1, 2, 4, 8, 8, 8])
        nv, kt = (16, 128) if dtype == "fp8" else (8, 64)
        M = max(1, round(_log_uniform(rng, 16, 16384)))
        if op not in ("gemm_rs_cols", "ag_gemm_k"):
            M = _multiple(M, P)                                   # rows are what is scattered or gathered
        hidden, inner = _log_uniform(rng, 256, 16384), _log_uniform(rng, 256, 8192)
        layout, act, slots, overlap = "kn", "none", "f32", False
        if op.startswith("ag"):
            N, K = P * _multiple(inner, nv), _multiple(hidden, kt * (P if op == "ag_gemm_k" else 1))
            act = rng.choice(["none", "relu", "gelu_tanh", "silu"])
            if op == "ag_gemm":
                layout = rng.choice(["kn", "nk"])
        else:
            N, K = _multiple(hidden, nv * (P if op == "gemm_rs_cols" else 1)), P * _multiple(inner, kt)
            if op == "gemm_rs":
                overlap = rng.random() < 0.5
                layout = rng.choice(["kn", "kn", "nk"])
            if layout == "kn":
                slots = rng.choice(["f32", "f32", "bf16"])
        c = _case(None, op, P, rng.randrange(P), M, N, K, dtype, layout, act, slots, overlap)
        if _cost(c) <= most:
            return c


# ---------------------------------------------------------------------------------------------------------------------
def _local(c):
    """(m, n, k) of this rank's GEMM, and (rows, columns) of one partial slot."""
    P, M, N, K = c["P"], c["M"], c["N"], c["K"]
    if c["op"].startswith("ag"):
        return (M, N // P, K), None
    return (M, N, K // P), ((M, N // P) if c["op"] == "gemm_rs_cols" else (M // P, N))


def _quantised(x, dtype):
    if dtype == "bf16":
        return x.bfloat16(), None
    scale = (x.abs().amax() / 448.0).reshape(1)
    return (x / scale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn), scale


def _inputs(c, seed):
    """Operands z/sqrt(K) with z ~ N(0,1), rounded to bf16 or quantised with one scale; peers' partial sums with the standard
    deviation that a partial sum of such operands has, and their reduced rows (all-reduce) with that of a whole sum."""
    (m, n, k), slot = _local(c)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    A, sa = _quantised(normal(m, k) / math.sqrt(c["K"]), c["dtype"])
    B, sb = _quantised(normal(k, n) / math.sqrt(c["K"]), c["dtype"])
    d = {"A": A, "B": B.t().contiguous() if c["layout"] == "nk" else B, "sa": sa, "sb": sb}
    if slot:
        part = normal(c["P"], *slot) * (math.sqrt(c["K"] / c["P"]) / c["K"])
        part[c["rank"]] = 0.0
        d["partials"] = part.bfloat16() if c["slots"] == "bf16" else part
    if c["op"] == "gemm_ar":
        d["rows"] = (normal(c["M"], c["N"]) / math.sqrt(c["K"])).bfloat16()
    return d


def prepare(case, seed):
    c, s = case, _inputs(case, seed)
    (m, n, k), slot = _local(c)
    P, rank = c["P"], c["rank"]
    s.update(case=c, epoch=0, status=torch.zeros(8, dtype=torch.int32, device="cuda"))

    def flags(*shape):
        f = torch.full(shape, READY, dtype=torch.int32, device="cuda")
        f[rank] = 0
        return f

    if slot is None:
        s["chunk_flags"] = flags(P)
        s["C"] = torch.zeros((m, n), dtype=torch.bfloat16, device="cuda")
        return s
    plan = getattr(pk, "pk_%s_plan" % c["op"])(P, c["M"], c["N"], c["K"], c["dtype"])
    s["flags_in"] = flags(P, plan.flags_per_slot)
    s["flags_out"] = torch.zeros_like(s["flags_in"])
    s["outgoing"] = torch.zeros_like(s["partials"])
    if c["op"] == "gemm_ar":
        s["full"] = s.pop("rows")
        s["bcast"] = torch.zeros((P, *slot), dtype=torch.bfloat16, device="cuda")
        s["ar_in"] = flags(P, plan.ar_flags_per_slot)
        s["ar_out"] = torch.zeros_like(s["ar_in"])
    else:
        s["out"] = torch.zeros(slot, dtype=torch.bfloat16, device="cuda")
    return s


def run(state):
    s, c = state, state["case"]
    s["epoch"] += 1
    P, rank = c["P"], c["rank"]
    head = (P, rank, c["M"], c["N"], c["K"], c["dtype"], s["A"], s["B"], s["sa"], s["sb"])
    if c["op"] == "ag_gemm":
        pk.pk_ag_gemm(*head, s["chunk_flags"], s["epoch"], s["C"], s["status"], act=c["act"], b_layout=c["layout"])
        return {"C": s["C"]}
    if c["op"] == "ag_gemm_k":
        pk.pk_ag_gemm_k(*head, s["chunk_flags"], s["epoch"], s["C"], s["status"], act=c["act"])
        return {"C": s["C"]}
    sent = {"own": s["partials"][rank], "outgoing": s["outgoing"]}
    slots = (s["partials"], s["outgoing"], s["flags_in"], s["flags_out"])
    if c["op"] == "gemm_ar":
        pk.pk_gemm_ar(*head, *slots, s["full"], s["bcast"], s["ar_in"], s["ar_out"], s["epoch"], pk.PHASE_ALL | pk.PHASE_WAIT,
                      s["status"], partial_dtype=c["slots"])
        return {"full": s["full"], "bcast": s["bcast"], **sent}
    if c["op"] == "gemm_rs_cols":
        pk.pk_gemm_rs_cols(*head, *slots, s["epoch"], s["out"], pk.PHASE_ALL, s["status"], partial_dtype=c["slots"])
    else:
        pk.pk_gemm_rs(*head, *slots, s["epoch"], s["out"], pk.PHASE_ALL | (pk.PHASE_OVERLAP if c["overlap"] else 0), s["status"],
                      partial_dtype=c["slots"], b_layout=c["layout"])
    return {"out": s["out"], **sent}


def work(case):
    c = case
    (m, n, k), slot = _local(c)
    elem = 1 if c["dtype"] == "fp8" else 2
    total = (m * k + k * n) * elem
    if slot is None:
        total += m * n * 2
    else:
        e, size = 2 if c["slots"] == "bf16" else 4, slot[0] * slot[1]
        # read: the peers' slots; written: this rank's product (own and outgoing slots) and the reduced rows, which the
        # all-reduce hands to every rank
        total += (c["P"] - 1) * size * e + m * n * e + size * 2 * (c["P"] if c["op"] == "gemm_ar" else 1)
    return {"bytes": total, "flops": 2 * m * n * k}


def tolerance(case):
    # bf16 results, correctly rounded: 1.7e-3 (2-norm) and at most half a unit in the last place, 2^-8 of the value, off the
    # 64-bit result; two correct implementations may round a value to neighbours, one unit apart
    return {"rel": 7e-3, "max": 1.6e-2}


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    P, rank = c["P"], c["rank"]
    (m, n, k), slot = _local(c)
    B = d["B"].t() if c["layout"] == "nk" else d["B"]
    x = d["A"].float().double() @ B.float().double().contiguous()
    if d["sa"] is not None:
        x *= d["sa"].double() * d["sb"].double()
    if slot is None:
        if c["act"] == "relu":
            x = x.clamp_min(0.0)
        elif c["act"] == "gelu_tanh":
            x = 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))
        elif c["act"] == "silu":
            x = x / (1.0 + torch.exp(-x))
        return {"C": x}
    if c["op"] == "gemm_rs_cols":
        own = x.reshape(c["M"], P, slot[1]).permute(1, 0, 2).contiguous()
    else:
        own = x.reshape(P, *slot)
    mine, outgoing = own[rank].clone(), own
    outgoing[rank] = 0.0                                          # no tile of the own block is sent
    out = mine.clone()
    for p in range(P):
        if p != rank:
            out += d["partials"][p].double()
    sent = {"own": mine, "outgoing": outgoing}
    if c["op"] != "gemm_ar":
        return {"out": out, **sent}
    full = d["rows"].double()
    full[rank * slot[0]:(rank + 1) * slot[0]] = out
    bcast = out.repeat(P, 1, 1)
    bcast[rank] = 0.0
    return {"full": full, "bcast": bcast, **sent}
