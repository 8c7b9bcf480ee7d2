"""pk_gemm_rs with PK_PHASE_OVERLAP (the reduce beside the second part of the GEMM, on the library's own stream):
parity against the float64 oracle and bit-identity with the plain call, on shapes whose schedule has more rounds than
the own block takes (so that the two-launch path is really taken, which is checked) and on some where the flag must fall back."""
import numpy as np
import pytest
import torch

from oracle import codec
from paper_2511_13940_amd import pk, workloads as wl
from tests import harness as hz
from tests.test_gpu_bf16_slots import check as check16
from tests.test_gpu_gemm_rs import check_rs

pytestmark = pytest.mark.gpu

OVERLAP = pk.PHASE_ALL | pk.PHASE_OVERLAP

CASES = [
    # P, rank, M, N, K, dtype, the plan's tile, tiles of the two launches (0: the flag is ignored, all tiles run at once)
    (8, 3, 4096, 2048, 2048, "bf16", 128, (256, 0)),
    (8, 7, 8192, 4096, 4096, "bf16", 256, (256, 256)),       # last rank: the row rotation wraps around
    (4, 1, 4400, 2056, 1024, "bf16", 128, (162, 0)),         # ragged
    (8, 2, 8192, 4096, 8192, "fp8", 256, (256, 256)),        # 256x256 fp8 kernel: the narrow reduce kernel runs beside it
    (4, 3, 8192, 4096 + 272, 4096, "fp8", 256, (504, 72)),   # the same with a ragged last column tile
    (2, 0, 4096, 8192, 1024, "bf16", 256, (256, 256)),       # own block = half of all tiles, two rounds of four
    (8, 3, 8 * 250, 8208, 8 * 256, "bf16", 128, (132, 396)),     # 128x256 tiles, blocks of two flag rows, the second ragged
    (8, 7, 8 * 200, 12304, 8 * 128, "bf16", 128, (196, 196)),    # 256x256 tiles over flags of 128x128, blocks of 200 rows
    (8, 5, 8 * 250, 8208, 8 * 256, "fp8", 128, (132, 396)),      # fp8 128x256 tiles beside the narrow reduce kernel
    (3, 1, 12288, 4128, 3 * 256, "fp8", 256, (476, 340)),        # 194 MiB of slots, P = 3: the run-time-P reduce beside the fp8 kernel
]


def launches(*args, **kw):
    r = hz.route("gemm_rs", *args, phases=OVERLAP, **kw)
    return r.first, r.second


@pytest.mark.parametrize("P,rank,M,N,K,dtype,tile,parts", CASES)
@pytest.mark.parametrize("deliver", ["pre", "emu"])
def test_overlapped_reduce_matches_oracle_and_plain_call(P, rank, M, N, K, dtype, tile, parts, deliver):
    assert launches(P, rank, M, N, K, dtype) == parts
    inp = wl.gemm_rs_inputs(P, M, N, K, dtype, rank, seed=11)
    kw = dict(scale_a=inp.get("scale_a"), scale_b=inp.get("scale_b"), deliver=deliver, order=inp["order"], epoch=5,
              timeout_us=2_000_000)
    plain = hz.run_gemm_rs(P, rank, M, N, K, dtype, inp["A_local"], inp["B_local"], inp["partials"], **kw)
    over = hz.run_gemm_rs(P, rank, M, N, K, dtype, inp["A_local"], inp["B_local"], inp["partials"], phases=OVERLAP, **kw)
    assert over["plan"].tile_m == tile
    check_rs(P, rank, dtype, inp, over, K // P)
    assert np.array_equal(over["out_bits"], plain["out_bits"])
    for q in range(P):
        if q != rank:
            assert np.array_equal(over["outgoing"][q].view(np.uint32), plain["outgoing"][q].view(np.uint32)), q
    assert np.array_equal(over["partials_after"][rank].view(np.uint32), plain["partials_after"][rank].view(np.uint32))
    assert np.array_equal(over["flags_out"], plain["flags_out"]) and np.array_equal(over["flags_in"], plain["flags_in"])


def test_flag_falls_back_when_the_own_block_takes_every_round():
    """One round in all (cfg1-sized problem): the call runs as the plain one does."""
    c = wl.CONFIGS["cfg1"]
    inp = wl.gemm_rs_inputs(c.P, c.M, c.N, c.K, c.dtype, 1, seed=2)
    res = hz.run_gemm_rs(c.P, 1, c.M, c.N, c.K, c.dtype, inp["A_local"], inp["B_local"], inp["partials"], phases=OVERLAP)
    check_rs(c.P, 1, c.dtype, inp, res, c.K // c.P)


@pytest.mark.parametrize("P,rank,M,N,K,parts", [
    (8, 4, 4096, 2048, 2048, (256, 0)),
    (8, 4, 4096, 8192, 2048, (256, 256)),                    # 256x256 tiles
    (8, 6, 8 * 250, 8208, 8 * 256, (132, 396)),              # 128x256 tiles
])
def test_bf16_slots_and_repeated_calls_with_rising_epochs(P, rank, M, N, K, parts):
    """bf16 partial slots next to the bf16 kernel, three calls in a row on the same buffers (the second stream and its
    events are reused; every call's reduce must see that call's own block)."""
    assert launches(P, rank, M, N, K, "bf16", partial_dtype="bf16") == parts
    outs = []
    for seed, epoch in ((1, 1), (2, 2), (1, 3)):
        inp = wl.gemm_rs_inputs(P, M, N, K, "bf16", rank, seed=seed)
        p16 = wl.to_bf16_bits(inp["partials"])
        res = hz.run_gemm_rs(P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], p16, epoch=epoch, phases=OVERLAP,
                             partial_dtype="bf16")
        ref = hz.run_gemm_rs(P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], p16, epoch=epoch, partial_dtype="bf16")
        assert res["status"][0] == 0 and ref["status"][0] == 0
        check16(P, rank, "bf16", dict(inp, partials16=p16), res, K // P)
        assert np.array_equal(res["out_bits"], ref["out_bits"])
        outs.append(res["out_bits"])
    assert np.array_equal(outs[0], outs[2]) and not np.array_equal(outs[0], outs[1])


def test_overlap_flag_needs_both_phases():
    t = torch.zeros(4096, dtype=torch.int32, device="cuda")
    for phases in (pk.PHASE_GEMM | pk.PHASE_OVERLAP, pk.PHASE_REDUCE | pk.PHASE_OVERLAP, pk.PHASE_OVERLAP):
        with pytest.raises(pk.PkError) as e:
            pk.pk_gemm_rs(2, 0, 256, 256, 512, "bf16", t, t, None, None, t, t, t, t, 1, t, phases, t)
        assert e.value.code == pk.ERR_ARG


def test_overlap_on_a_compute_unit_partition_with_live_peers():
    """The GEMM launches on the compute stream of a partition (224 workgroups), the peers' partials arrive through the
    communicator stream while it runs, the reduce on the library's own stream: same bits as the plain pre-landed call."""
    P, rank, M, N, K = 4, 3, 4096, 4096, 4 * 256
    assert launches(P, rank, M, N, K, "bf16", comm_cus=32) == (192, 64)
    inp = wl.gemm_rs_inputs(P, M, N, K, "bf16", rank, seed=21)
    base = hz.run_gemm_rs(P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], inp["partials"])
    check_rs(P, rank, "bf16", inp, base, K // P)
    comp, comm = pk.pk_partition_create(32)
    try:
        for i, n_wg in enumerate([32, 128]):
            order = wl.arrival_order(P, rank, "random", seed=i)
            res = hz.run_gemm_rs(P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], inp["partials"], deliver="emu",
                                 order=order, epoch=i + 1, comm_cus=32, n_wg=n_wg, partition=(comp, comm), phases=OVERLAP,
                                 timeout_us=2_000_000)
            assert res["status"][0] == 0
            assert np.array_equal(res["out_bits"], base["out_bits"])
            for q in range(P):
                if q != rank:
                    assert np.array_equal(res["outgoing"][q].view(np.uint32), base["outgoing"][q].view(np.uint32))
    finally:
        torch.cuda.synchronize()
        pk.pk_partition_destroy(comp, comm)


def test_overlap_flag_with_a_single_rank_is_the_plain_gemm():
    inp = wl.gemm_rs_inputs(1, 1024, 2048, 512, "bf16", 0, seed=4)
    res = hz.run_gemm_rs(1, 0, 1024, 2048, 512, "bf16", inp["A_local"], inp["B_local"], inp["partials"], phases=OVERLAP)
    check_rs(1, 0, "bf16", inp, res, 512)


@pytest.mark.parametrize("dtype,M,N,K,parts", [
    ("bf16", 8192, 4096, 8192, (256, 256)),                  # the narrow reduce kernel beside the k-contiguous GEMM kernel
    ("fp8", 8192, 4096, 8192, (512, 0)),                     # less than 192 MiB of slots: the flag is ignored
    ("fp8", 16384, 4096, 8 * 256, (256, 768)),               # 256 MiB: the narrow reduce kernel beside the k-contiguous fp8 kernel
])
def test_overlap_flag_with_a_k_contiguous_second_operand(dtype, M, N, K, parts):
    P, rank = 8, 6
    assert launches(P, rank, M, N, K, dtype, b_layout="nk") == parts
    inp = wl.gemm_rs_inputs(P, M, N, K, dtype, rank, seed=13)
    Bt = np.ascontiguousarray(inp["B_local"].T)
    kw = dict(scale_a=inp.get("scale_a"), scale_b=inp.get("scale_b"), epoch=3)
    plain = hz.run_gemm_rs(P, rank, M, N, K, dtype, inp["A_local"], inp["B_local"], inp["partials"], **kw)
    over = hz.run_gemm_rs(P, rank, M, N, K, dtype, inp["A_local"], Bt, inp["partials"], phases=OVERLAP, b_layout="nk", **kw)
    assert over["plan"].tile_m == 256
    check_rs(P, rank, dtype, inp, over, K // P)
    assert np.array_equal(over["out_bits"], plain["out_bits"])


# Sizes at which both launches of the call are more than one round of workgroups with a partial last one, the condition for a
# stream-K tail when a launch stands alone.
@pytest.mark.parametrize("P,rank,M,N,K,dtype,comm_cus", [
    (4, 1, 4096, 4352, 4 * 1024, "bf16", 192),        # 64 workgroups: 204 + 68 tiles
    (8, 0, 8192, 6144, 8192, "bf16", 0),              # 480 + 288 tiles
    (3, 2, 12288, 5120, 6144, "fp8", 0),              # 480 + 480 tiles
])
def test_overlapped_reduce_with_a_workspace(P, rank, M, N, K, dtype, comm_cus):
    """The two launches must not meet in the workspace: the same bits as the plain call without one, three calls with rising epochs
    on one workspace, which stays the call site's own (a plain call with it follows)."""
    assert all(t > (256 - comm_cus) and t % (256 - comm_cus) for t in launches(P, rank, M, N, K, dtype, comm_cus=comm_cus, workspace=True))
    inp = wl.gemm_rs_inputs(P, M, N, K, dtype, rank, seed=15)
    kw = dict(scale_a=inp.get("scale_a"), scale_b=inp.get("scale_b"), comm_cus=comm_cus)
    args = (P, rank, M, N, K, dtype, inp["A_local"], inp["B_local"], inp["partials"])
    plain = hz.run_gemm_rs(*args, epoch=1, **kw)
    if M * N * K // P < 2 ** 36:
        check_rs(P, rank, dtype, inp, plain, K // P)
    ws = torch.zeros(plain["plan"].workspace_bytes // 4, dtype=torch.int32, device="cuda")
    for epoch in (1, 2, 3):
        over = hz.run_gemm_rs(*args, epoch=epoch, phases=OVERLAP, workspace=ws, **kw)
        assert over["status"][0] == 0
        assert np.array_equal(over["out_bits"], plain["out_bits"]), epoch
        assert np.array_equal(over["partials_after"][rank].view(np.uint32), plain["partials_after"][rank].view(np.uint32)), epoch
        for q in range(P):
            if q != rank:
                assert np.array_equal(over["outgoing"][q].view(np.uint32), plain["outgoing"][q].view(np.uint32)), (epoch, q)
    tail = hz.run_gemm_rs(*args, epoch=4, workspace=ws, **kw)
    assert tail["status"][0] == 0
    # another order of the same fp32 sums: neighbouring bf16 values at most
    a, b = codec.bf16_decode(tail["out_bits"]), codec.bf16_decode(plain["out_bits"])
    assert np.max(np.abs(a - b) / (np.abs(b) + 1.0)) <= 1e-2


def test_a_workspace_too_small_for_either_launch_is_refused_before_anything_runs():
    P, rank, M, N, K = 4, 1, 4096, 4352, 4 * 1024
    inp = wl.gemm_rs_inputs(P, M, N, K, "bf16", rank, seed=16)
    with pytest.raises(pk.PkError) as e:
        hz.run_gemm_rs(P, rank, M, N, K, "bf16", inp["A_local"], inp["B_local"], inp["partials"], phases=OVERLAP, comm_cus=192,
                       workspace=torch.zeros(2048, dtype=torch.int32, device="cuda"))
    assert e.value.code == pk.ERR_ARG
