"""GPU parity of pk_ag_gemm against the float64 oracle, through the C ABI.

Gate: max |gpu - ref| / (|ref| + 1) <= 1e-2 (bf16 inputs), <= 5e-2 (fp8).  Derived bound: fp32
accumulation of k products (2*k*2^-24 * sum|a||b|) plus half a bf16 ulp of the result (2^-8 relative)."""
import itertools

import numpy as np
import pytest
import torch

from oracle import codec, tp_gemm
from paper_2511_13940_amd import pk, workloads as wl
from tests import harness as hz

pytestmark = pytest.mark.gpu

GATE = {"bf16": 1e-2, "fp8": 5e-2}
U32 = 2.0 ** -24


def gate_err(gpu, ref):
    return float(np.max(np.abs(gpu - ref) / (np.abs(ref) + 1.0)))


def check_ag(P, rank, dtype, inp, res, K):
    A = tp_gemm.gather_chunks(inp["chunks"])
    ref = tp_gemm.ag_gemm(P, rank, A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    mag = tp_gemm.abs_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    assert res["status"][0] == 0, res["status"]
    got = codec.bf16_decode(res["C_bits"])
    assert not np.isnan(got).any()
    assert gate_err(got, ref["C"]) <= GATE[dtype]
    bound = 2 * K * U32 * mag + 2.0 ** -8 * np.abs(ref["C"]) + 2.0 ** -133
    assert np.all(np.abs(got - ref["C"]) <= bound)
    return ref


@pytest.mark.parametrize("rank", [0, 1, 2, 3])
def test_cfg2_every_rank(rank):
    c = wl.CONFIGS["cfg2"]
    inp = wl.ag_gemm_inputs(c.P, c.M, c.N, c.K, c.dtype, rank, seed=0, order="random")
    res = hz.run_ag_gemm(c.P, rank, c.M, c.N, c.K, c.dtype, inp["chunks"], inp["B_local"], epoch=3)
    check_ag(c.P, rank, c.dtype, inp, res, c.K)


def test_cfg2_all_arrival_orders_bitwise_identical_and_no_early_reads():
    """All 6 orders of the 3 peer chunks, delivered by the emulator into NaN-poisoned rows while the
    GEMM runs: the output is bit-identical to the pre-landed run (and so contains no NaN)."""
    c = wl.CONFIGS["cfg2"]
    rank = 1
    inp = wl.ag_gemm_inputs(c.P, c.M, c.N, c.K, c.dtype, rank, seed=1)
    base = hz.run_ag_gemm(c.P, rank, c.M, c.N, c.K, c.dtype, inp["chunks"], inp["B_local"])
    check_ag(c.P, rank, c.dtype, inp, base, c.K)
    full = tp_gemm.gather_chunks(inp["chunks"])
    peers = [q for q in range(c.P) if q != rank]
    for i, order in enumerate(itertools.permutations(peers)):
        res = hz.run_ag_gemm(c.P, rank, c.M, c.N, c.K, c.dtype, inp["chunks"], inp["B_local"],
                             deliver="emu", order=list(order), gap_us=(0, 40, 200)[i % 3], epoch=i + 1)
        assert res["status"][0] == 0
        assert np.array_equal(res["C_bits"], base["C_bits"]), f"order {order}"
        assert np.array_equal(res["A_after"].view(np.uint16), full)       # A_gathered == concat of the chunks
        assert np.all(res["flags"][peers] == i + 1)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("P,M,N,K,rank", [
    (2, 2 * 200, 2 * 136, 256, 1),     # ragged rows per chunk and ragged columns (N/P = 136)
    (4, 4 * 96, 4 * 272, 384, 3),      # chunk smaller than a tile, 3 column tiles with a 16-wide tail
    (1, 384, 256, 128, 0),             # P = 1: plain GEMM, no flags
    (3, 3 * 128, 3 * 128, 512, 2),
])
def test_ragged_small_tiles(dtype, P, M, N, K, rank):
    if dtype == "fp8" and ((N // P) % 16 or K % 128):
        pytest.skip("shape not valid for fp8")
    inp = wl.ag_gemm_inputs(P, M, N, K, dtype, rank, seed=2)
    res = hz.run_ag_gemm(P, rank, M, N, K, dtype, inp["chunks"], inp["B_local"], inp["scale_a"], inp["scale_b"])
    check_ag(P, rank, dtype, inp, res, K)


@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("ragged", [False, True])
def test_big_tiles(dtype, ragged):
    """256 x 256 tiles: 4 chunks x 4 tile rows x 16 tile columns = 256 tiles; emulated ring arrival."""
    P, rank = 4, 2
    M = 4 * (1024 - (24 if ragged else 0))
    N = 4 * (4096 - (80 if ragged else 0))
    K = 256
    assert pk.pk_ag_gemm_plan(P, M, N, K, dtype).tile_m == 256
    inp = wl.ag_gemm_inputs(P, M, N, K, dtype, rank, seed=4)
    res = hz.run_ag_gemm(P, rank, M, N, K, dtype, inp["chunks"], inp["B_local"], inp["scale_a"], inp["scale_b"],
                         deliver="emu", order=inp["order"], gap_us=20)
    check_ag(P, rank, dtype, inp, res, K)


def test_column_shards_concatenate_to_the_full_product():
    P, M, N, K = 4, 512, 1024, 256
    g = wl.global_problem(M, N, K, "bf16", seed=6)
    chunks = [wl.slice_ag_gemm(g, P, q)[0] for q in range(P)]
    cols = []
    for r in range(P):
        res = hz.run_ag_gemm(P, r, M, N, K, "bf16", chunks, wl.slice_ag_gemm(g, P, r)[1])
        assert res["status"][0] == 0
        cols.append(codec.bf16_decode(res["C_bits"]))
    full = tp_gemm.local_product(g["A"], g["B"], "bf16")
    got = np.concatenate(cols, axis=1)
    assert gate_err(got, full) <= GATE["bf16"]
    assert np.all(np.abs(got - full) <= 2.0 ** -8 * np.abs(full) + 1e-5)


def test_missing_chunk_times_out_instead_of_hanging():
    P, rank, M, N, K = 4, 0, 512, 512, 128
    inp = wl.ag_gemm_inputs(P, M, N, K, "bf16", rank, seed=8)
    res = hz.run_ag_gemm(P, rank, M, N, K, "bf16", inp["chunks"], inp["B_local"], epoch=5, withhold=2,
                         timeout_us=2000)
    assert res["status"][0] == pk.ERR_TIMEOUT and res["status"][1] == 2 and res["status"][2] == 1
    ref = tp_gemm.ag_gemm(P, rank, tp_gemm.gather_chunks(inp["chunks"]), inp["B_local"], "bf16")["C"]
    got = codec.bf16_decode(res["C_bits"])
    mp = M // P
    keep = np.r_[0:2 * mp, 3 * mp:M]
    assert gate_err(got[keep], ref[keep]) <= GATE["bf16"]          # the other chunks' tiles were computed
    assert np.all(res["C_bits"][2 * mp:3 * mp] == 0xFFFF)          # the withheld chunk's rows were left alone


@pytest.mark.parametrize("act", ["relu", "gelu_tanh", "silu"])
@pytest.mark.parametrize("dtype,P,M,N,K,rank", [
    ("bf16", 2, 2 * 200, 2 * 264, 256, 1),      # ragged 128-tiles
    ("bf16", 2, 4096, 2 * 2048, 256, 0),        # 256-tiles
    ("fp8", 2, 512, 2 * 256, 256, 1),
])
def test_fused_activation(act, dtype, P, M, N, K, rank):
    """act(A.B) in the epilogue: fp32 evaluation on the accumulator, then one rounding to bf16.  The inputs are scaled up
    so that the pre-activations spread over a few units (the non-linear range)."""
    inp = wl.ag_gemm_inputs(P, M, N, K, dtype, rank, seed=31)
    if dtype == "bf16":          # x 16 on one operand: exact in bf16, pre-activations ~ N(0, 1)
        inp["B_local"] = codec.bf16_encode(codec.bf16_decode(inp["B_local"]) * 16.0)
    res = hz.run_ag_gemm(P, rank, M, N, K, dtype, inp["chunks"], inp["B_local"], inp["scale_a"], inp["scale_b"], act=act)
    assert res["status"][0] == 0
    A = tp_gemm.gather_chunks(inp["chunks"])
    ref = tp_gemm.ag_gemm(P, rank, A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"], act=act)["C"]
    mag = tp_gemm.abs_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    got = codec.bf16_decode(res["C_bits"])
    assert not np.isnan(got).any()
    assert gate_err(got, ref) <= GATE[dtype]
    # the activations are 1.13-Lipschitz: the accumulation error passes through at most that much amplified; the fp32
    # evaluation of exp / tanh adds a few fp32 ulps of the result and of x
    pre = tp_gemm.ag_gemm(P, rank, A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])["C"]
    bound = 1.13 * 2 * K * U32 * mag + 2.0 ** -8 * np.abs(ref) + 16 * U32 * (np.abs(pre) + 1.0) + 2.0 ** -133
    assert np.all(np.abs(got - ref) <= bound)
    if act == "relu":
        assert np.all(got >= 0) and np.any(got == 0) and np.any(got > 0)


@pytest.mark.parametrize("act,lowest", [("silu", -88.5), ("gelu_tanh", -10.0)])
@pytest.mark.parametrize("K", [64, 4096])                   # 32 x 32 tiles; 256 x 128 or larger with 4200 rows
def test_activation_of_every_bf16_value(act, lowest, K):
    """x * 1 is exact, so every row holds the activation of one bf16 value, down to results near the smallest normal number.  Both
    are x / (1 + exp(-y)), with y = x or GELU's inner polynomial (in this form, since 1 + tanh() cancels in float64 as well).
    Bound: half a bf16 ulp, and in units of 2^-24 of the value 4 for the exponential, the sum and the quotient and, for GELU, the
    five roundings of y and its constants, which the exponential turns into 5 |y|."""
    bits = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)
    x = codec.bf16_decode(bits)
    x = x[np.isfinite(x) & (np.abs(x) >= 2.0 ** -10) & (x >= lowest) & (x <= 88.5)]
    M, N = x.size, 2048 if K > 64 else 8
    A = np.zeros((M, K), dtype=np.uint16)
    A[:, K - 1] = codec.bf16_encode(x)
    B = np.zeros((K, N), dtype=np.uint16)
    B[K - 1, :] = 0x3F80                                      # 1.0
    res = hz.run_ag_gemm(1, 0, M, N, K, "bf16", [A], B, act=act)
    assert res["status"][0] == 0
    y = x if act == "silu" else 2 * np.sqrt(2 / np.pi) * (x + 0.044715 * x ** 3)
    want, units = (x / (1 + np.exp(-y)))[:, None], (4 + (0 if act == "silu" else 5) * np.abs(y))[:, None]
    got = codec.bf16_decode(res["C_bits"])
    assert np.all(np.abs(got - want) <= (2.0 ** -8 + units * 2.0 ** -24) * np.abs(want) + 2.0 ** -134)


@pytest.mark.parametrize("act", ["silu", "gelu_tanh", "relu"])
def test_activation_of_special_values(act):
    """Infinities, NaN, the largest values and zeros among ordinary ones: x * sigmoid(y) is NaN at -infinity (0 times infinity), zero
    with its sign for large negative values, x for large positive ones; max(x, 0) takes no NaN."""
    x = np.array([np.inf, -np.inf, np.nan, 3e38, -3e38, 1e4, -1e4, 0.0, -0.0, 1.5, 88.0, -200.0])
    relu = act == "relu"
    want = np.array([np.inf, 0.0 if relu else np.nan, 0.0 if relu else np.nan, 3e38, 0.0, 1e4, 0.0, 0.0, 0.0, np.nan, 88.0, 0.0])
    M, N, K = 96, 16, 64
    A, B = np.zeros((M, K), dtype=np.uint16), np.zeros((K, N), dtype=np.uint16)
    A[:, 0] = np.resize(codec.bf16_encode(np.where(np.isfinite(x), x, 0.0)), M)
    A[:, 0] = np.where(np.resize(x, M) == np.inf, 0x7F80, np.where(np.resize(x, M) == -np.inf, 0xFF80, A[:, 0]))
    A[np.isnan(np.resize(x, M)), 0] = 0x7FC0
    B[0, :] = 0x3F80
    res = hz.run_ag_gemm(1, 0, M, N, K, "bf16", [A], B, act=act)
    got = codec.bf16_decode(res["C_bits"])
    for i in range(M):
        w = want[i % x.size]
        if i % x.size == 9:
            w = tp_gemm.activation(1.5, act)                  # an ordinary value beside the special ones
        assert np.all(np.isnan(got[i]) if np.isnan(w) else np.isclose(got[i], w, rtol=2.0 ** -8, atol=0)), (i, x[i % x.size], got[i, 0])


def test_mlp_block_chain_matches_the_oracle():
    """AG + GEMM with fused SiLU, its bf16 output fed to GEMM + RS as the local operand (paper section 4.1), against the
    oracle's chained definition."""
    P, rank, M, D, I = 4, 1, 2048, 1024, 4096
    rng_seed = 41
    inp1 = wl.ag_gemm_inputs(P, M, I, D, "bf16", rank, seed=rng_seed)                       # X chunks, W1[:, I_rank]: D x I/P
    inp1["B_local"] = codec.bf16_encode(codec.bf16_decode(inp1["B_local"]) * 16.0)
    inp2 = wl.gemm_rs_inputs(P, M, D, I, "bf16", rank, seed=rng_seed + 1)                   # W2[I_rank, :]: I/P x D, peers' partials
    h = hz.run_ag_gemm(P, rank, M, I, D, "bf16", inp1["chunks"], inp1["B_local"], act="silu")
    assert h["status"][0] == 0
    res = hz.run_gemm_rs(P, rank, M, D, I, "bf16", h["C_bits"], inp2["B_local"], inp2["partials"])
    assert res["status"][0] == 0
    X = tp_gemm.gather_chunks(inp1["chunks"])
    ref = tp_gemm.mlp_block(P, rank, X, inp1["B_local"], inp2["B_local"], inp2["partials"], act="silu")
    # H: a few elements may round to the neighbouring bf16 value (fp32 vs float64 evaluation next to a tie)
    hg, hr = codec.bf16_decode(h["C_bits"]), codec.bf16_decode(ref["H_bf16"])
    assert np.mean(h["C_bits"] != ref["H_bf16"]) < 0.02
    mag1 = tp_gemm.abs_product(X, inp1["B_local"], "bf16")
    assert np.all(np.abs(hg - hr) <= 1.13 * 2 * D * U32 * mag1 + 2.0 ** -7 * np.abs(hr) + 2.0 ** -133)
    got = codec.bf16_decode(res["out_bits"])
    assert gate_err(got, ref["out"]) <= GATE["bf16"]
    # second GEMM on the GPU's own H: exact parity chain (no tie ambiguity)
    ref2 = tp_gemm.gemm_rs(P, rank, h["C_bits"], inp2["B_local"], "bf16", inp2["partials"])
    mag = tp_gemm.abs_product(h["C_bits"], inp2["B_local"], "bf16")
    mp = M // P
    slot_mag = np.abs(ref2["outgoing"][rank]) + sum(np.abs(inp2["partials"][q].astype(np.float64)) for q in range(P) if q != rank)
    bound = 2 * (I // P) * U32 * mag[rank * mp:(rank + 1) * mp] + P * U32 * slot_mag + 2.0 ** -8 * np.abs(ref2["out"]) + 2.0 ** -133
    assert np.all(np.abs(got - ref2["out"]) <= bound)


def test_chunks_delivered_by_copies_and_stream_flag_writes():
    """Chunks moved by device-to-device copies with a stream memory operation per flag (no communicator workgroups),
    into poisoned rows while the GEMM runs on every compute unit: bit-identical to the pre-landed run."""
    c = wl.CONFIGS["cfg2"]
    rank = 3
    inp = wl.ag_gemm_inputs(c.P, c.M, c.N, c.K, c.dtype, rank, seed=2)
    base = hz.run_ag_gemm(c.P, rank, c.M, c.N, c.K, c.dtype, inp["chunks"], inp["B_local"])
    check_ag(c.P, rank, c.dtype, inp, base, c.K)
    full = tp_gemm.gather_chunks(inp["chunks"])
    for i, order in enumerate([[0, 1, 2], [2, 0, 1]]):
        res = hz.run_ag_gemm(c.P, rank, c.M, c.N, c.K, c.dtype, inp["chunks"], inp["B_local"], deliver="dma",
                             order=order, epoch=i + 1)
        assert res["status"][0] == 0
        assert np.array_equal(res["C_bits"], base["C_bits"])
        assert np.array_equal(res["A_after"].view(np.uint16), full)
        assert np.all(res["flags"][order] == i + 1)


def test_ten_seeded_arrival_orders_of_seven_chunks_bitwise_identical():
    """P = 8: ten seeded permutations of the 7 peer chunks with different gaps, delivered into poisoned rows while the
    GEMM runs (each workgroup meets several chunks): bit-identical to the pre-landed run, no NaN."""
    P, rank, M, N, K = 8, 3, 8 * 256, 8 * 128, 256
    inp = wl.ag_gemm_inputs(P, M, N, K, "bf16", rank, seed=61)
    base = hz.run_ag_gemm(P, rank, M, N, K, "bf16", inp["chunks"], inp["B_local"])
    check_ag(P, rank, "bf16", inp, base, K)
    for s in range(10):
        order = wl.arrival_order(P, rank, "random", seed=100 + s)
        res = hz.run_ag_gemm(P, rank, M, N, K, "bf16", inp["chunks"], inp["B_local"], deliver="emu", order=order,
                             gap_us=(0, 20, 120)[s % 3], epoch=s + 1, fetch_A=False)
        assert res["status"][0] == 0
        assert np.array_equal(res["C_bits"], base["C_bits"]), f"order {order}"


def test_chunk_memory_read_by_another_kernel_before_the_chunk_lands():
    """A kernel on a third stream reads what the buffer held before (NaN) while the call computes on other chunks, so that lines of
    it are in the L2s when the chunks land; they land before the call's first look at them (its second round of tiles).  What
    counts is memory at the time of the flag: the same bits as with all chunks in place."""
    P, rank, M, n, K = 4, 1, 4096, 7168, 8192             # 448 tiles of 256 x 256: two rounds of some 180 us
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    full = (torch.randn(M, K, generator=g, device="cuda") / K ** 0.5).bfloat16()
    B = (torch.randn(K, n, generator=g, device="cuda") / K ** 0.5).bfloat16()
    status = torch.zeros(8, dtype=torch.int32, device="cuda")
    counters = torch.zeros(pk.EMU_MAX_ORDER, dtype=torch.int32, device="cuda")
    flags = torch.full((P,), 1, dtype=torch.int32, device="cuda")
    want, C = (torch.zeros((M, n), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    pk.pk_ag_gemm(P, rank, M, P * n, K, "bf16", full, B, None, None, flags, 1, want, status)
    mp = M // P
    A = torch.empty_like(full)
    feeder, reader = torch.cuda.Stream(), torch.cuda.Stream()
    order = [(rank + d) % P for d in range(1, P)]
    for epoch, gap in ((2, 40), (3, 60), (4, 20)):
        A.fill_(float("nan"))
        A[rank * mp:(rank + 1) * mp] = full[rank * mp:(rank + 1) * mp]
        counters.zero_()
        C.zero_()
        torch.cuda.synchronize()
        pk.pk_emu_deliver_chunks(P, M, K, 2, full, A, flags, epoch, order, gap, counters, stream=feeder)
        pk.pk_ag_gemm(P, rank, M, P * n, K, "bf16", A, B, None, None, flags, epoch, C, status, comm_cus=32)
        with torch.cuda.stream(reader):
            seen = [A[q * mp:(q + 1) * mp].clone() for q in order[1:]]
        torch.cuda.synchronize()
        assert status[0].item() == 0
        assert torch.equal(C.view(torch.int16), want.view(torch.int16)), epoch
        del seen
