"""Every tile shape of the GEMM kernels at the sizes where it can go wrong: ragged rows and columns, k ranges shorter and longer
than the load ring, tiles that cover several ready flags or several chunks, and flags published behind the GEMM (tiles finer
than a flag).  The tile shape that each size leads to (chosen by estimated time, csrc/pk_tiles.h) stands beside it and is checked
here and, without a GPU, in test_routes.py.

Bounds as in test_gpu_gemm_rs.py: fp32 accumulation of k products in any order, 2*k*2^-24 * sum|a||b|, and half a bf16 ulp."""
import numpy as np
import pytest
import torch

from oracle import codec, tp_gemm
from paper_2511_13940_amd import pk, workloads as wl
from tests import harness as hz
from tests.test_gpu_bf16_slots import check as check_rs16
from tests.test_gpu_gemm_rs import check_rs

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


# dtype, P, rank, M, N, K/P, layout of the second operand, slots, (tile, flags published behind the GEMM) of the whole call and of
# its GEMM phase as a call of its own
RS_CASES = [
    ("bf16", 8, 3, 1024, 4104, 2560, "kn", "f32", "256x128", "256x128"),      # two flags per tile, the last column tile 8 wide
    ("bf16", 2, 1, 2800, 4104, 128, "kn", "f32", "256x256", "256x256"),       # four flags per tile, shards of 11 flag rows (odd)
    ("bf16", 8, 5, 8 * 96, 8200, 512, "nk", "f32", "128x256 late", "128x256 late"),   # over shards of 96 rows
    ("bf16", 5, 4, 5 * 300, 1544, 128, "kn", "f32", "128x128 late", "128x128"),       # late: tiles cross shards of 300 rows
    ("bf16", 4, 0, 2048, 1024, 448, "nk", "f32", "128x64 late", "128x128"),   # finer than a flag, seven k-tiles in a ring of four
    ("bf16", 2, 1, 700, 1480, 832, "kn", "f32", "128x64 late", "128x128"),    # 13 k-tiles
    ("bf16", 8, 2, 8 * 77, 1040, 1152, "kn", "f32", "64x64 late", "128x128"), # 18 k-tiles; tiles cross shards of 77 rows
    ("fp8", 2, 0, 520, 1552, 256, "kn", "f32", "64x64 late", "128x128"),      # two k-tiles in a ring of six
    ("bf16", 4, 2, 4 * 75, 1000, 1088, "nk", "f32", "32x64 late", "32x64 late"),      # shards of 75 rows, 17 k-tiles over four waves
    ("bf16", 2, 1, 256, 248, 64, "kn", "f32", "32x32 late", "128x256"),       # one k-tile, three of the four waves without work
    ("bf16", 8, 7, 64, 520, 4032, "kn", "f32", "32x32 late", "32x32 late"),   # shards of 8 rows, 63 k-tiles
    ("bf16", 3, 1, 6000, 5008, 512, "kn", "f32", "256x256", "256x256"),       # two rounds; rows that start on 64 bytes: each tile's stores are waited for
    ("bf16", 2, 1, 5124, 4840, 320, "kn", "f32", "256x256", "256x256"),       # the same, rows that start on 32 bytes
    ("fp8", 2, 0, 4600, 8208, 512, "kn", "f32", "256x256", "256x256"),        # the same, 64 bytes and three rounds (on 128: test_gpu_k_ranges.py)
    ("fp8", 8, 2, 8 * 33, 4112, 256, "kn", "f32", "128x64 late", "128x128"),
    ("fp8", 2, 0, 2000, 4112, 256, "nk", "f32", "256x256", "256x256"),        # shards of 1000 rows
    ("fp8", 3, 2, 3 * 500, 2064, 2176, "kn", "f32", "128x128", "128x128"),    # 17 k-tiles
    ("fp8", 1, 0, 130, 144, 1152, "kn", "f32", "32x32 late", "128x128"),      # nine k-tiles over four waves
    # fp32 rows that start on 128-byte lines (written in pieces of 32 columns; those of the cases above mostly do not)
    ("bf16", 8, 3, 1024, 4128, 2560, "kn", "f32", "256x128", "256x128"),
    ("bf16", 8, 1, 6000, 1184, 320, "kn", "f32", "128x256 late", "128x256"),
    ("bf16", 8, 1, 6000, 1160, 320, "kn", "f32", "128x256 late", "128x256"),  # (not on lines)
    ("bf16", 8, 3, 1024, 4096, 2560, "kn", "f32", "128x128", "128x128"),
    ("bf16", 8, 2, 8 * 77, 1024, 1152, "kn", "f32", "64x64 late", "128x128"),
    ("bf16", 4, 2, 4 * 75, 992, 1088, "nk", "f32", "32x64 late", "32x64 late"),
    ("bf16", 8, 7, 64, 512, 4032, "kn", "f32", "32x32 late", "32x32 late"),
    ("fp8", 8, 2, 8 * 33, 4096, 256, "kn", "f32", "128x64 late", "128x128"),
    ("fp8", 2, 0, 520, 1536, 256, "kn", "f32", "64x64 late", "128x128"),
    ("bf16", 8, 3, 1024, 4104, 2560, "kn", "bf16", "256x128", "256x128"),     # bf16 slots from here on
    ("bf16", 8, 2, 8 * 77, 1040, 1152, "kn", "bf16", "64x64 late", "128x128"),
    ("bf16", 8, 7, 64, 520, 4032, "kn", "bf16", "32x32 late", "32x32 late"),
    ("bf16", 3, 1, 6000, 5008, 512, "kn", "bf16", "256x256", "256x256"),
    ("fp8", 2, 0, 520, 1552, 256, "kn", "bf16", "64x64 late", "128x128"),
    ("fp8", 8, 2, 8 * 33, 4112, 256, "kn", "bf16", "128x64 late", "128x128"),
    ("fp8", 2, 0, 4600, 8208, 512, "kn", "bf16", "256x256", "256x256"),
]


def tile(op, *args, **kw):
    r = hz.route(op, *args, **kw)
    return r.tile + (" late" if r.late else "")


@pytest.mark.parametrize("dtype,P,rank,M,N,kl,layout,slots,whole,alone", RS_CASES)
def test_gemm_rs(dtype, P, rank, M, N, kl, layout, slots, whole, alone):
    kw = dict(partial_dtype=slots, b_layout=layout)
    assert tile("gemm_rs", P, rank, M, N, P * kl, dtype, **kw) == whole
    assert tile("gemm_rs", P, rank, M, N, P * kl, dtype, phases=pk.PHASE_GEMM, **kw) == alone
    inp = wl.gemm_rs_inputs(P, M, N, P * kl, dtype, rank, seed=M + N)
    B = np.ascontiguousarray(inp["B_local"].T) if layout == "nk" else inp["B_local"]
    inp["partials16"] = wl.to_bf16_bits(inp["partials"])
    args = (P, rank, M, N, P * kl, dtype, inp["A_local"], B, inp["partials16" if slots == "bf16" else "partials"], inp["scale_a"],
            inp["scale_b"])
    # the whole call, and its phases as calls of their own (which may use other tiles and so add in another order)
    for epoch, phases in ((6, pk.PHASE_ALL), (9, (pk.PHASE_GEMM, pk.PHASE_REDUCE))):
        res = hz.run_gemm_rs(*args, epoch=epoch, phases=phases, **kw)
        (check_rs16 if slots == "bf16" else check_rs)(P, rank, dtype, inp, res, kl)
        assert np.all(res["flags_in"][rank] == epoch) and all(np.all(res["flags_out"][q] == epoch) for q in range(P) if q != rank)
        assert P == 1 or np.all(res["flags_out"][rank] == 0)
    # every flag is out before a reduce is launched
    g = hz.run_gemm_rs(*args, epoch=12, phases=pk.PHASE_GEMM, **kw)
    assert np.all(g["flags_in"][rank] == 12) and all(np.all(g["flags_out"][q] == 12) for q in range(P) if q != rank)


COLS_CASES = [
    (4, 1, 1000, 8192, 256, "bf16", "128x256"),          # inside column blocks of 2048
    (4, 2, 333, 4 * 1032, 128, "bf16", "128x64 late"),   # column blocks of 1032
    (2, 0, 1500, 2 * 2064, 128, "fp8", "128x256"),       # the last tile of a column block 16 wide
]


@pytest.mark.parametrize("P,rank,M,N,kl,dtype,want_tile", COLS_CASES)
def test_gemm_rs_cols(P, rank, M, N, kl, dtype, want_tile):
    assert tile("gemm_rs_cols", P, rank, M, N, P * kl, dtype) == want_tile
    inp = wl.gemm_rs_inputs(P, M * P, N, P * kl, dtype, rank, seed=M)
    A = np.ascontiguousarray(inp["A_local"][:M])
    partials = (np.random.default_rng(M).standard_normal((P, M, N // P)) * 0.02).astype(np.float32)
    res = hz.run_gemm_rs(P, rank, M, N, P * kl, dtype, A, inp["B_local"], partials, inp["scale_a"], inp["scale_b"], epoch=4, cols=True)
    assert res["status"][0] == 0
    ref = tp_gemm.gemm_rs_cols(P, rank, A, inp["B_local"], dtype, partials, inp["scale_a"], inp["scale_b"])
    mag = tp_gemm.abs_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    ns = N // P
    # the 8-bit MFMA adds the 64 products of one instruction with an error of up to 2^-14 of the largest of them (see
    # test_gpu_special_values.py); 448 is the largest code
    mfma8 = (kl // 64) * 2.0 ** -14 * 448.0 ** 2 * inp["scale_a"] * inp["scale_b"] if dtype == "fp8" else 0.0
    for q in range(P):
        got = res["partials_after"][rank] if q == rank else res["outgoing"][q]
        assert np.all(np.abs(got - ref["outgoing"][q]) <= 2 * kl * U32 * mag[:, q * ns:(q + 1) * ns] + mfma8 + 1e-30), q
        assert q == rank or np.all(res["flags_out"][q] == 4)


AG_CASES = [
    ("bf16", 8, 2, 1024, 8 * 4104, 2560, "kn", "none", "256x128"),        # one tile covers two chunks of 128 rows
    ("bf16", 3, 1, 2100, 3 * 2056, 192, "nk", "relu", "128x256"),         # chunks of 700 rows
    ("bf16", 8, 6, 8 * 189, 8 * 1720, 576, "kn", "silu", "128x128"),      # across chunks of 189 rows
    ("bf16", 4, 3, 1000, 4 * 1544, 320, "nk", "gelu_tanh", "128x64"),
    ("bf16", 64, 40, 64 * 3, 64 * 72, 1024, "kn", "none", "32x32"),       # 64 chunks of 3 rows: a tile waits for ten and more of them
    ("bf16", 2, 0, 6000, 2 * 1800, 64, "kn", "silu", "256x256"),
    ("bf16", 2, 1, 9000, 2 * 2312, 256, "kn", "gelu_tanh", "128x256"),    # three rounds, chunk by chunk
    ("bf16", 2, 1, 7200, 2 * 3600, 256, "kn", "gelu_tanh", "256x256"),    # two rounds, chunk by chunk; inner tiles and ragged edges
    ("bf16", 3, 2, 6000, 3 * 4112, 192, "kn", "none", "256x256"),         # the same with too few k-tiles for stores to drain under
    ("fp8", 2, 0, 7200, 2 * 4112, 512, "kn", "silu", "256x256"),
    ("bf16", 8, 3, 64, 8 * 1000, 2048, "kn", "silu", "32x32"),
    ("bf16", 4, 3, 4 * 25, 4 * 4000, 320, "nk", "none", "32x64"),         # five k-tiles over four waves
    ("bf16", 2, 0, 2 * 150, 2 * 2064, 1152, "kn", "gelu_tanh", "64x64"),
    ("fp8", 4, 1, 4 * 75, 4 * 2064, 640, "nk", "relu", "64x64"),
    ("fp8", 8, 0, 24, 8 * 3600, 896, "kn", "none", "32x32"),              # seven k-tiles
    ("fp8", 5, 2, 5 * 77, 5 * 1040, 640, "kn", "gelu_tanh", "32x64"),
    ("fp8", 8, 7, 2048, 8 * 3600, 256, "nk", "silu", "128x256"),
]


@pytest.mark.parametrize("dtype,P,rank,M,N,K,layout,act,want_tile", AG_CASES)
def test_ag_gemm(dtype, P, rank, M, N, K, layout, act, want_tile):
    assert tile("ag_gemm", P, rank, M, N, K, dtype, b_layout=layout) == want_tile
    inp = wl.ag_gemm_inputs(P, M, N, K, dtype, rank, seed=M + N)
    B = np.ascontiguousarray(inp["B_local"].T) if layout == "nk" else inp["B_local"]
    runs = [hz.run_ag_gemm(P, rank, M, N, K, dtype, inp["chunks"], B, inp["scale_a"], inp["scale_b"], epoch=3, act=act,
                           b_layout=layout, deliver=d, order=inp["order"]) for d in ("pre", "emu")]
    A = tp_gemm.gather_chunks(inp["chunks"])
    x = tp_gemm.local_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    mag = tp_gemm.abs_product(A, inp["B_local"], dtype, inp["scale_a"], inp["scale_b"])
    want = tp_gemm.activation(x, act)
    for res in runs:
        assert res["status"][0] == 0
        got = codec.bf16_decode(res["C_bits"])
        # the slope of every activation is at most 1.13; the fp32 evaluation adds a few units of 2^-23
        assert np.all(np.abs(got - want) <= 1.13 * 2 * K * U32 * mag + (2.0 ** -8 + 2.0 ** -20) * np.abs(want) + 2.0 ** -133)
    assert np.array_equal(runs[0]["C_bits"], runs[1]["C_bits"])   # whatever arrives when


def test_ag_gemm_chunks_that_share_a_cache_line():
    """A_gathered starts 16 bytes into a 128-byte line, so the last line of a chunk holds the first bytes of the next one."""
    P, rank, M, N, K = 4, 1, 4 * 48, 4 * 264, 128
    inp = wl.ag_gemm_inputs(P, M, N, K, "bf16", rank, seed=5)
    full = hz.dev(tp_gemm.gather_chunks(inp["chunks"]).view(np.int16))
    mem = torch.full((M * K + 64,), 0x7FC1, dtype=torch.int16, device="cuda")
    A = mem[8:8 + M * K].view(M, K)
    assert A.data_ptr() % 128 == 16
    A[rank * 48:(rank + 1) * 48] = full[rank * 48:(rank + 1) * 48]
    B = hz.elem_view(inp["B_local"], "bf16")
    C = torch.zeros((M, N // P), dtype=torch.int16, device="cuda")
    flags = torch.zeros(P, dtype=torch.int32, device="cuda")
    status = torch.zeros(8, dtype=torch.int32, device="cuda")
    counters = torch.zeros(pk.EMU_MAX_ORDER, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    pk.pk_emu_deliver_chunks(P, M, K, 2, full, A, flags, 1, [3, 0, 2], 5, counters, stream=side)
    pk.pk_ag_gemm(P, rank, M, N, K, "bf16", A, B, None, None, flags, 1, C, status)
    torch.cuda.synchronize()
    assert status[0].item() == 0
    A_bits = tp_gemm.gather_chunks(inp["chunks"])
    want = tp_gemm.local_product(A_bits, inp["B_local"], "bf16")
    mag = tp_gemm.abs_product(A_bits, inp["B_local"], "bf16")
    assert np.all(np.abs(codec.bf16_decode(hz.bits_of(C)) - want) <= 2 * K * U32 * mag + 2.0 ** -8 * np.abs(want) + 2.0 ** -133)


AGK_CASES = [
    ("bf16", 4, 2, 999, 4 * 2056, 4 * 64, "128x128"),    # one k-tile per chunk
    ("bf16", 8, 5, 1500, 8 * 640, 8 * 192, "64x64"),
    ("fp8", 2, 1, 300, 2 * 528, 2 * 384, "64x64"),       # three k-tiles per chunk
]


@pytest.mark.parametrize("dtype,P,rank,M,N,K,want_tile", AGK_CASES)
def test_ag_gemm_k(dtype, P, rank, M, N, K, want_tile):
    assert tile("ag_gemm_k", P, rank, M, N, K, dtype) == want_tile
    g = wl.global_problem(M, N, K, dtype, seed=M)
    kp, ns = K // P, N // P
    chunks = [np.ascontiguousarray(g["A"][:, q * kp:(q + 1) * kp]) for q in range(P)]
    B = np.ascontiguousarray(g["B"][:, rank * ns:(rank + 1) * ns])
    runs = [hz.run_ag_gemm_k(P, rank, M, N, K, dtype, chunks, B, g["scale_a"], g["scale_b"], epoch=2, deliver=d) for d in ("pre", "dma")]
    want = tp_gemm.local_product(g["A"], B, dtype, g["scale_a"], g["scale_b"])
    mag = tp_gemm.abs_product(g["A"], B, dtype, g["scale_a"], g["scale_b"])
    for res in runs:
        assert res["status"][0] == 0
        got = codec.bf16_decode(res["C_bits"])
        assert np.all(np.abs(got - want) <= 2 * K * U32 * mag + 2.0 ** -8 * np.abs(want) + 2.0 ** -133)
    # all chunks there from the start, or one by one: the k range is summed in the same order
    assert np.array_equal(runs[0]["C_bits"], runs[1]["C_bits"])


def test_a_workspace_changes_nothing_where_the_plan_has_128x128_tiles():
    """288 flag tiles of 128 x 128: the same bits with and without a workspace, and one that is too small is refused."""
    P, rank, M, N, K = 2, 1, 2304, 2048, 2 * 1024
    inp = wl.gemm_rs_inputs(P, M, N, K, "bf16", rank, seed=9)
    plan = pk.pk_gemm_rs_plan(P, M, N, K, "bf16")
    assert plan.tile_m == 128 and P * plan.tiles_m * plan.tiles_n > 256
    assert not hz.route("gemm_rs", P, rank, M, N, K, "bf16", workspace=True).stream_k
    args = (P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], inp["partials"])
    plain, with_ws = hz.run_gemm_rs(*args), hz.run_gemm_rs(*args, workspace=True)
    assert np.array_equal(plain["out_bits"], with_ws["out_bits"])
    assert np.array_equal(plain["outgoing"][1 - rank], with_ws["outgoing"][1 - rank])
    with pytest.raises(pk.PkError) as e:
        hz.run_gemm_rs(*args, workspace=torch.zeros(4096, dtype=torch.int32, device="cuda"))
    assert e.value.code == pk.ERR_ARG


def test_overlap_flag_beside_the_fp8_kernel_with_bf16_slots():
    """256 MiB of slots: the wide reduce kernel beside the second part of the GEMM (with less the flag is ignored there)."""
    P, rank, M, N, K = 8, 5, 16384, 8192, 8 * 128
    inp = wl.gemm_rs_inputs(P, M, N, K, "fp8", rank, seed=10)
    p16 = wl.to_bf16_bits(inp["partials"])
    args = (P, rank, M, N, K, "fp8", inp["A_local"], inp["B_local"], p16, inp["scale_a"], inp["scale_b"])
    assert hz.route("gemm_rs", P, rank, M, N, K, "fp8", phases=pk.PHASE_ALL | pk.PHASE_OVERLAP, partial_dtype="bf16").second > 0
    plain = hz.run_gemm_rs(*args, partial_dtype="bf16")
    over = hz.run_gemm_rs(*args, partial_dtype="bf16", phases=pk.PHASE_ALL | pk.PHASE_OVERLAP)
    assert plain["status"][0] == 0 and over["status"][0] == 0
    assert np.array_equal(over["out_bits"], plain["out_bits"])
    for q in range(P):
        assert q == rank or np.array_equal(over["outgoing"][q], plain["outgoing"][q])


@pytest.mark.parametrize("P,rank,M,N,kl", [(4, 1, 1600, 376, 256), (8, 7, 64, 520, 4032)])
def test_flags_published_behind_the_gemm_do_not_wait_for_a_late_peer(P, rank, M, N, kl):
    """One flag of one peer never comes: that tile's reduce gives up after the time limit, but every flag of this rank's own work is
    out, also those of that tile (other ranks wait for them)."""
    assert hz.route("gemm_rs", P, rank, M, N, P * kl, "bf16").late
    inp = wl.gemm_rs_inputs(P, M, N, P * kl, "bf16", rank, seed=3)
    res = hz.run_gemm_rs(P, rank, M, N, P * kl, "bf16", inp["A_local"], inp["B_local"], inp["partials"], epoch=5, timeout_us=20000,
                         withhold=((rank + 1) % P, 0))
    assert res["status"][0] == pk.ERR_TIMEOUT and res["status"][1] == 0 and res["status"][2] == 2
    assert np.all(res["flags_in"][rank] == 5)
    assert all(np.all(res["flags_out"][q] == 5) for q in range(P) if q != rank)
